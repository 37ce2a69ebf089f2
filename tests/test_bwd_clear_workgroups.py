"""Host-only check (no GPU) of the workgroups that clear what a packed backward call leaves out of dBm and dCm: as many as a long, mostly unused axis
needs, few for a short one."""
import ctypes
import os

import pytest

from paper_2602_08810_amd import api

LIB = os.path.join(os.path.dirname(api.__file__), "liblrnnx.so")


def test_share_of_a_workgroup():
    if not os.path.exists(LIB):
        pytest.skip("liblrnnx.so not built")
    count = ctypes.CDLL(LIB)._ZN5lrnnx13bwd_clear_wgsEli         # lrnnx::bwd_clear_wgs(L, floats of a row)
    for floats in (1, 2, 4, 8, 16, 32):
        for L in (1, 100, 4097, 16384, 65537, 131072, 1 << 20, 1 << 31):
            wgs = count(ctypes.c_int64(L), floats)
            assert 16 <= wgs <= 512 and (wgs == 512 or L * floats < 2 * 8192 * wgs), (L, floats, wgs)
            assert wgs == 16 or wgs * 8192 <= L * floats
