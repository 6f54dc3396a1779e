"""What the lane kernel's wavefronts share in a workgroup (mcs_team.h), on the
CPU: nodes of a stopped unit are handed in once, whoever leaves last, and a
workgroup is counted as idle once, whoever says so; and which records it takes
(record_fits, mcs_layout.h)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def _run(tmp_path, name):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs g++")
    exe = str(tmp_path / name)
    r = subprocess.run([gxx, "-O1", "-std=c++17", "-pthread", "-I",
                        os.path.join(ROOT, "paper_1908_06418_amd", "csrc"),
                        os.path.join(HERE, "lane_model", name + ".cpp"), "-o", exe],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-4000:]
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60)
    return r.returncode, r.stdout


def test_transitions_of_a_team(tmp_path):
    code, out = _run(tmp_path, "team")
    assert code == 0 and "orders 384 bad 0 idle 0" in out, out


def test_records_that_are_taken_fit(tmp_path):
    code, out = _run(tmp_path, "record")
    assert code == 0, out


def test_launch_parameters_fit_their_place_in_lds(tmp_path):
    code, out = _run(tmp_path, "params")
    assert code == 0, out
