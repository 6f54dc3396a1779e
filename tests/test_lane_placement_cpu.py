"""Where the kernel with a search in every lane puts its frames, replayed on
the CPU (tests/lane_model/placement.cpp, with the library's own rule): a lane's
part of the stack holds what does not enter the wavefront's worst-case area,
and one search at a time is in that area."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("lane_model") / "placement")
    r = subprocess.run([gxx, "-O2", "-std=c++17", "-I",
                        os.path.join(ROOT, "paper_1908_06418_amd", "csrc"),
                        os.path.join(HERE, "lane_model", "placement.cpp"), "-o", exe],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-4000:]
    return exe


# bits, n, p, labels per vertex, pairs, node limit, cap: the library's caps
# where the stacks pass them, and the smallest cap (one frame of n classes),
# where many lanes want the area at once
@pytest.mark.parametrize("case", [(64, 64, 0.1, 0.5, 30, 200_000, 160),
                                  (128, 124, 0.1, 0.75, 10, 200_000, 256),
                                  (64, 64, 0.1, 0.5, 2, 20_000, 65),
                                  (32, 32, 0.2, 0.3, 20, 100_000, 34)])
def test_one_search_at_a_time_in_the_worst_case_area(model, case):
    r = subprocess.run([model] + [str(x) for x in case], stdout=subprocess.PIPE, text=True,
                       timeout=300)
    assert r.returncode == 0, r.stdout
    words = r.stdout.split()
    got = dict(zip(words[::2], map(int, words[1::2])))
    print(got)
    # children that start where the lane's part ends, lanes that had to wait
    assert got["at_cap"] > 0 and got["entered"] > 0 and got["waited"] > 0
    assert got["bad"] == 0
