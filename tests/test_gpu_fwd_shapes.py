"""GPU parity of the forward pass at the edges of a lane, a checkpoint interval and a tile, with outputs, last state and every
checkpoint, whatever shape the launch rule takes; the shapes over several tiles are in test_gpu_fwd_tiles.py."""
import numpy as np
import pytest

from paper_2602_08810_amd import workloads
from _util import TOL, check_outputs, dev, host, sel_inputs_dev

pytestmark = pytest.mark.gpu

DISCS = ["zoh_s6", "zoh", "bilinear", "dirac"]


@pytest.fixture(scope="module")
def api():
    from paper_2602_08810_amd import api as _api
    _api.lib()
    return _api


# Odd channel counts leave lanes and wavefronts of the last workgroup without a channel; N = 32 stages its maps twice.
@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("N,B,D,L", [
    (16, 1, 2501, 17), (32, 1, 2301, 255), (1, 1, 3001, 256), (2, 1, 2601, 100), (8, 2, 4201, 257), (16, 2, 4501, 511),
    (16, 2, 11, 511), (32, 1, 9, 257), (1, 1, 3, 9), (4, 1, 2, 8), (8, 3, 13, 512),
    (16, 1, 9, 1025), (32, 1, 5, 1023), (2, 1, 3, 1024), (4, 2, 17, 2049)])
def test_forward_shapes(api, oracle, io, N, B, D, L):
    disc = DISCS[(N + D + L) % 4]
    p = workloads.make_selective(B=B, D=D, N=N, L=L, io=io, gate=True, with_x0=True, seed=N + L, bias=("uniform", -4.0, -2.0))
    y, x, ckpt = api.lrnnx_selective_scan_fwd(**sel_inputs_dev(p, io), disc=disc, return_last_state=True, return_ckpt=True)
    ref = {k: p[k] for k in ("u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "x0")}
    yr, xr, xs = oracle.selective_scan_fwd(disc=disc, return_states=True, **ref)
    before = np.concatenate([p["x0"][:, :, None, :], xs[:, :, 255:L - 1:256, :]], axis=2)     # states entering 0, 256, ...
    check_outputs({"y": (host(y), yr, TOL[io]), "x_last": (host(x), xr, 1e-4), "ckpt": (host(ckpt), before, 1e-4)}, disc)


# chunks of one tile each
@pytest.mark.parametrize("N,L", [(16, 255), (16, 257), (32, 1025), (4, 2000), (1, 513)])
def test_forward_chunks(api, oracle, N, L):
    p = workloads.make_selective(B=2, D=21, N=N, L=L, io="f32", gate=True, with_x0=True, seed=L, bias=("uniform", -4.0, -2.0))
    y, x = api.lrnnx_selective_scan_fwd(**sel_inputs_dev(p, "f32"), return_last_state=True, path="chunk_carry")
    yr, xr = oracle.selective_scan_fwd(**{k: p[k] for k in ("u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "x0")})
    check_outputs({"y": (host(y), yr, 1e-4), "x_last": (host(x), xr, 1e-4)})


# packed batches: many rows of short sequences 16 lanes (bfloat16); else 64 lanes, of 4 steps, of 8 or of 16 as the sequences get
# longer
@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("N,D,lengths", [
    (4, 2101, (1, 255, 256, 257, 7, 300)), (16, 11, (1, 3, 256, 257, 1030, 515)), (2, 1025, (2047, 2100)), (8, 9, (4097, 5121))])
def test_forward_packed_shapes(api, oracle, io, N, D, lengths):
    import torch
    p = workloads.make_packed(D=D, N=N, lengths=lengths, io=io, seed=N)
    t = {k: dev(p[k], io) for k in ("u", "delta", "Bm", "Cm", "z")}
    t.update({k: dev(p[k]) for k in ("A", "Dskip", "delta_bias", "x0")})
    y, x = api.lrnnx_selective_scan_fwd(**t, cu_seqlens=torch.from_numpy(p["cu_seqlens"]).cuda(), return_last_state=True)
    ref = {k: p[k] for k in ("u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "x0")}
    yr, xr = oracle.selective_scan_fwd_packed(cu_seqlens=p["cu_seqlens"], **ref)
    check_outputs({"y": (host(y), yr, TOL[io]), "x_last": (host(x), xr, 1e-4)})
