"""The binding takes the address of any numpy array, whatever its dtype, order
and flags (CPU; no GPU call)."""
import numpy as np
import pytest

from paper_1305_3345_amd import aesgpu


def read_only():
    a = np.arange(7, dtype=np.uint8)
    a.flags.writeable = False
    return a


@pytest.mark.parametrize("a", [
    np.zeros(5, "M8[s]"), np.zeros(5, "m8[ns]"), np.zeros(2, [("t", "M8[s]"), ("n", "u4")]),
    np.zeros(3, "V0"), np.zeros(3, "V5"), np.zeros(3, object), np.zeros(3, "U4"),
    np.zeros(4, ">u8"), np.zeros(4, np.float16), np.zeros((), np.uint8), np.zeros(0, np.uint8),
    np.zeros((6, 4))[::2], np.zeros((6, 4), order="F"), np.arange(9)[::-1], read_only(),
    np.zeros(3, aesgpu.REQ_DTYPE), np.zeros(3, aesgpu.REQ_DTYPE)["length"]], ids=str)
def test_address(a):
    assert aesgpu._ptr(a) == a.ctypes.data
