"""GPU parity at the ends of sequences: lengths around the steps a thread takes at once (1 to 16) and around a tile, as rows
of a larger allocation whose gaps hold NaN (nothing past the end may reach a result) and as packed neighbours."""
import numpy as np
import pytest

from paper_2602_08810_amd import workloads
from _util import TOL, check_outputs, dev, host, sel_inputs_dev

pytestmark = pytest.mark.gpu

NAMES = ("du", "ddelta", "dz", "dA", "dBm", "dCm", "dD", "dbias", "dx0")


@pytest.fixture(scope="module")
def api():
    from paper_2602_08810_amd import api as _api
    _api.lib()
    return _api


def _gapped(t):
    """The same [B,D,L] tensor as rows of L + 24 elements, NaN in between."""
    import torch
    big = torch.full((*t.shape[:2], t.shape[2] + 24), float("nan"), dtype=t.dtype, device=t.device)
    big[:, :, :t.shape[2]] = t
    return big[:, :, :t.shape[2]]


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("N,D,L", [(1, 5, 1), (1, 5, 7), (1, 9, 259), (2, 5, 3), (2, 7, 263), (4, 5, 2), (4, 9, 5), (4, 9, 257),
                                   (8, 5, 1), (8, 11, 300), (16, 5, 1), (16, 19, 9), (16, 19, 271), (32, 3, 17), (32, 5, 511)])
def test_rows_with_gaps(api, oracle, io, N, D, L):
    p = workloads.make_selective(B=2, D=D, N=N, L=L, io=io, gate=True, with_x0=True, seed=N + L, bias=("uniform", -4.0, -2.0))
    t, dy = sel_inputs_dev(p, io), _gapped(dev(p["dy"], io))
    for k in ("u", "delta", "z"):
        t[k] = _gapped(t[k])
    ref = {k: p[k] for k in ("u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "x0")}
    y, x, ckpt = api.lrnnx_selective_scan_fwd(**t, return_last_state=True, return_ckpt=True)
    g = api.lrnnx_selective_scan_bwd(**t, dy=dy, ckpt=ckpt, want_dx0=True)
    yr, xr = oracle.selective_scan_fwd(**ref)
    r = oracle.selective_scan_bwd(dy=p["dy"], **ref)
    check = {"y": (host(y), yr, TOL[io]), "x_last": (host(x), xr, 1e-4)}
    check.update({k: (host(g[k]), r[k], TOL[io] if k in ("du", "ddelta", "dz") else 1e-4) for k in NAMES})
    check_outputs(check)


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("N", [1, 2, 4, 8, 16, 32])
def test_packed_neighbours(api, oracle, io, N):
    import torch
    lengths = (1, 2, 3, 5, 7, 8, 9, 15, 16, 17, 33, 255, 256, 257, 263, 1)
    p = workloads.make_packed(D=11, N=N, lengths=lengths, io=io, seed=N)
    t = {k: dev(p[k], io) for k in ("u", "delta", "Bm", "Cm", "z")}
    t.update({k: dev(p[k]) for k in ("A", "Dskip", "delta_bias", "x0")})
    cu, dy = torch.from_numpy(p["cu_seqlens"]).cuda(), dev(p["dy"], io)
    ref = {k: p[k] for k in ("u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "x0")}
    y, x, ckpt = api.lrnnx_selective_scan_fwd(**t, cu_seqlens=cu, return_last_state=True, return_ckpt=True)
    g = api.lrnnx_selective_scan_bwd(**t, dy=dy, ckpt=ckpt, cu_seqlens=cu, max_seqlen=263, want_dx0=True)
    yr, xr = oracle.selective_scan_fwd_packed(cu_seqlens=p["cu_seqlens"], **ref)
    r = oracle.selective_scan_bwd_packed(dy=p["dy"], cu_seqlens=p["cu_seqlens"], **ref)
    check = {"y": (host(y), yr, TOL[io]), "x_last": (host(x), xr, 1e-4)}
    check.update({k: (host(g[k]), r[k], TOL[io] if k in ("du", "ddelta", "dz") else 1e-4) for k in NAMES})
    check_outputs(check)
