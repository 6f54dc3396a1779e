"""The kernel with a search in every lane is built, like the other search
kernels, without gfx950's three-input bitwise instruction."""
import os
import shutil
import subprocess

import pytest

from paper_1908_06418_amd import build


@pytest.mark.skipif(not os.path.exists(build.HIPCC) and shutil.which("hipcc") is None,
                    reason="hipcc not available")
def test_lane_kernel_has_no_bitop3(tmp_path):
    out = tmp_path / "mcs_lane.s"
    cmd = [build.HIPCC] + [f for f in build.COMMON if f != "-fPIC"] + [
        "--cuda-device-only", "-S", "-o", str(out), os.path.join(build.CSRC, "mcs_lane.hip")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    text = out.read_text()
    assert "mcs_lane_kernel" in text
    assert "v_bitop3" not in text
