"""Host-only checks of the launch shape of packed backward calls (no GPU): a workgroup never takes more channels than the kernel's tables in
LDS hold, 128 in the real pass and 64 in the complex one."""
import ctypes
import os
import random

import pytest

from paper_2602_08810_amd import api

LIB = os.path.join(os.path.dirname(api.__file__), "liblrnnx.so")


class Plan(ctypes.Structure):
    _fields_ = [("G", ctypes.c_int), ("nchunks", ctypes.c_int), ("tiles_per_chunk", ctypes.c_int64)]


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        pytest.skip("liblrnnx.so not built")
    return ctypes.CDLL(LIB)


# the library's own host functions (lrnnx:: in csrc/kernels.hpp): channels per workgroup as the entry point of a packed backward call has them
def _channels(lib, cplx, B, D, groups, N, L, longest):
    c = "c" if cplx else ""
    plan = getattr(lib, f"_ZN5lrnnx{8 + cplx}{c}bwd_planEiiilib")
    plan.restype = Plan
    shape = getattr(lib, f"_ZN5lrnnx{16 + cplx}{c}bwd_packed_shapeEiiiillPiS0_S0_")
    i64 = ctypes.c_int64
    G = ctypes.c_int(plan(B * groups, D // groups, N, i64(L), 1, False).G)       # a single pass over sequences of unknown lengths
    cap, fewest = ctypes.c_int(), ctypes.c_int()
    shape(B, D, groups, N, i64(L), i64(longest), ctypes.byref(G), ctypes.byref(cap), ctypes.byref(fewest))
    return G.value, cap.value, fewest.value


@pytest.mark.parametrize("cplx,most", [(False, 128), (True, 64)])
def test_channels_fit_the_tables(lib, cplx, most):
    r = random.Random(11)
    cases = [(32, 2560, 1, 16, 16384, 1200), (22, 2560, 1, 16, 12654, 1676), (32, 2048, 1, 16, 16071, 1603), (53, 2048, 1, 8, 22854, 996),
             (32, 2048, 1, 16, 8192, 512), (48, 1536, 1, 16, 32768, 2048)]
    for _ in range(20000):
        B, groups = r.randrange(2, 301), r.choice([1, 1, 1, 2, 4])
        D, L = groups * r.randrange(1, 5121 // groups), B * r.randrange(1, 3000)
        longest = r.choice([0, min(L, -(-L // B) * r.randrange(1, 9)), r.randrange(1, L + 1), 1, 2 * L])
        cases.append((B, D, groups, r.choice([1, 2, 4, 8, 16] + [32] * (not cplx)), L, longest))
    for case in cases:
        G, cap, fewest = _channels(lib, cplx, *case)
        assert 1 <= G <= most and (cap == 0 or 1 <= fewest <= G), (case, G, cap, fewest)
