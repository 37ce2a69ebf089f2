"""Host-only check (no GPU): the scratch that a real backward call asks for does not depend on the type of the rows, which callers of the size query
need not have set."""
import ctypes
import os
import random

import pytest

from paper_2602_08810_amd import api

LIB = os.path.join(os.path.dirname(api.__file__), "liblrnnx.so")


def test_size_is_the_same_for_both_types():
    if not os.path.exists(LIB):
        pytest.skip("liblrnnx.so not built")
    size = api.lib().lrnnx_selective_scan_bwd_workspace_bytes
    r = random.Random(3)
    for _ in range(20000):
        a = api.BwdArgs()
        a.struct_size = ctypes.sizeof(api.BwdArgs)
        a.N, a.bc_groups = r.choice([1, 2, 4, 8, 16, 32]), r.choice([1, 1, 2])
        a.B, a.D, a.L = int(2 ** r.uniform(0, 5)), int(2 ** r.uniform(0, 11)) * a.bc_groups, int(2 ** r.uniform(8, 19))
        need = []
        for a.io_dtype in (api.F32, api.BF16):
            need.append(int(size(ctypes.byref(a))))
        assert need[0] == need[1], (a.B, a.bc_groups, a.D, a.N, a.L, need)
