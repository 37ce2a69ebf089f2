"""Host-only checks of the scratch that a real backward call asks for (no GPU): bounded, enough for the plan that will run,
and never more than the general size query names."""
import ctypes
import os
import random

import pytest

from paper_2602_08810_amd import api

LIB = os.path.join(os.path.dirname(api.__file__), "liblrnnx.so")
MIB = 1 << 20
CAP = 512 * MIB + 512                                       # the tile sums of dBm and dCm, and what aligning them takes


@pytest.fixture(scope="module")
def call():
    if not os.path.exists(LIB):
        pytest.skip("liblrnnx.so not built")
    api.lib()

    def exact(B, D, N, L, ckpt=True, groups=1, packed=False, longest=0, path=0):
        a = api.BwdArgs()
        a.struct_size = ctypes.sizeof(api.BwdArgs)
        a.B, a.D, a.N, a.L, a.bc_groups, a.path, a.max_seqlen = B, D, N, L, groups, path, longest
        a.ckpt = 0x1000 if ckpt else None
        a.cu_seqlens = 0x1000 if packed else None
        return int(api.lib().lrnnx_selective_scan_bwd_workspace_bytes(ctypes.byref(a)))
    return exact


# (B, D, N, L, packed, longest): calls that took hundreds of megabytes to gigabytes of scratch for their tile sums
LARGE = [(16, 2560, 16, 4096, False, 0), (64, 2560, 16, 4096, False, 0), (1, 2048, 16, 65536, False, 0), (2, 2048, 16, 16384, False, 0),
         (8, 1536, 32, 16384, False, 0), (1, 768, 16, 1 << 20, False, 0),
         (96, 2560, 16, 131072, True, 0), (96, 2560, 16, 131072, True, 30000), (24, 5120, 16, 131072, True, 20000), (2, 2560, 16, 32768, True, 20000)]


@pytest.mark.parametrize("B,D,N,L,packed,longest", LARGE)
def test_sums_are_bounded(call, B, D, N, L, packed, longest):
    assert api.lrnnx_workspace_bytes(api.WS_BWD_SUMS, B, D, N, L, api.BF16, 1, packed) <= CAP
    need = call(B, D, N, L, packed=packed, longest=longest)
    nch = api.lib().lrnnx_selective_scan_bwd_chunks(B, D, N, L, 1, 0, 0)
    aggregates = 2 * B * D * N * 4 * (64 if packed else nch)
    assert need <= CAP + aggregates


def test_queries_agree(call):
    """Over random shapes the exact size covers the checkpoints and the chunks that run, and stays within the general query."""
    r = random.Random(5)
    for _ in range(3000):
        N, G = r.choice([1, 2, 4, 8, 16, 32]), r.choice([1, 1, 2, 3])
        D, B, L = r.randrange(1, 900) * G, int(2 ** r.uniform(0, 7)), int(2 ** r.uniform(0, 17))
        packed, ckpt, path = r.random() < 0.4, r.random() < 0.5, r.choice([0, 0, 1, 2])
        longest = r.choice([0, r.randrange(1, L + 1)]) if packed else 0
        need = call(B, D, N, L, ckpt, G, packed, longest, path)
        kinds = [api.WS_BWD_CARRY if ckpt else api.WS_BWD, api.WS_BWD_SUMS]
        general = sum(api.lrnnx_workspace_bytes(k, B, D, N, L, api.F32, G, packed) for k in kinds)
        assert need <= general, (B, D, N, L, G, packed, ckpt, path, longest)
        least = 0 if ckpt else (D * (L // 256 + B) if packed else B * D * -(-L // 256)) * N * 4
        if not packed:
            nch = api.lib().lrnnx_selective_scan_bwd_chunks(B, D, N, L, G, path, 0)
            least += 2 * B * D * nch * N * 4 if nch > 1 else 0
        assert need >= least


def test_invalid_calls_need_nothing(call):
    assert call(1, 8, 3, 100) == 0 and call(0, 8, 16, 100) == 0 and call(1, 9, 16, 100, groups=2) == 0
    assert call(1, 8, 16, 100, path=7) == 0 and call(70000, 8, 16, 100) == 0
    assert api.lib().lrnnx_selective_scan_bwd_workspace_bytes(None) == 0
    assert api.lib().lrnnx_selective_scan_bwd_workspace_bytes(ctypes.byref(api.BwdArgs())) == 0       # struct_size 0
