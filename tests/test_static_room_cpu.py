"""The static scratch against what one copy of the launch's counters per XCD
adds to a workspace: a batch that takes MCS_STATIC_SCRATCH_BYTES beside them
fits."""
import ctypes


def test_static_scratch_has_room_for_the_counters_of_each_xcd(mcs_lib):
    from paper_1908_06418_amd import _abi
    size, err = ctypes.c_size_t(0), ctypes.c_int(0)
    f = mcs_lib.mcs_internal_static_scratch
    f.restype = ctypes.c_void_p
    f(ctypes.byref(size), ctypes.byref(err))  # (the size does not need a device)
    # 8 copies of 128 bytes, and up to one more unit of 256 by rounding
    assert size.value >= _abi.MCS_STATIC_SCRATCH_BYTES + 8 * 128 + 256
