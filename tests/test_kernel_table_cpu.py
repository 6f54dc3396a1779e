"""The tables from which the plan takes its kernel: each gives its own kernels
and nothing else."""
import ctypes

import pytest


def _table(lib, name):
    f = getattr(lib, name)
    f.restype = ctypes.c_void_p
    f.argtypes = [ctypes.c_int] * 3
    return f


@pytest.mark.parametrize("word", [4, 8, 16, 32])
@pytest.mark.parametrize("directed", [0, 1])
def test_segment_table_has_segment_kernels_only(mcs_lib, word, directed):
    seg = _table(mcs_lib, "mcs_internal_seg_kernel")
    lane = _table(mcs_lib, "mcs_internal_lane_kernel")
    for log in range(-2, 8):
        assert (seg(word, directed, log) is not None) is (word <= 8 and log in (2, 3, 4))
    lanes = {lane(word, directed, 0), lane(word, directed, 1)}
    assert lane(word, directed, 0) is not None
    assert (lane(word, directed, 1) is not None) is (word <= 8)
    assert not lanes & {seg(word, directed, log) for log in (2, 3, 4)} or word > 8
