"""GPU parity of the forward kernel's four shapes walking several tiles with a ragged last one: the state carried from tile to
tile, the fetch of the next tile, and the step from whole tiles to a part of one, for every N and I/O type and with the
discretisations in turn; and the chunked path where a chunk has several tiles."""
import pytest

from paper_2602_08810_amd import workloads
from _util import TOL, check_outputs, dev, host, sel_inputs_dev

pytestmark = pytest.mark.gpu

DISCS = ["zoh_s6", "zoh", "bilinear", "dirac"]
NS = [1, 2, 4, 8, 16, 32]
# shape: {N: (channels, steps)} of one batch entry for which the launch rule takes that shape, with both I/O types (16 lanes for
# N <= 2: with bfloat16; float32 takes 64 lanes of 4 steps there)
SHAPES = {
    "16 lanes": {N: (8191, 700) for N in NS},
    "64 lanes, 4 steps": {1: (5, 1100), 2: (5, 1100), 4: (9, 1100), 8: (5, 1100), 16: (5, 700), 32: (9, 700)},
    "64 lanes, 8 steps": {1: (2051, 1300), 2: (2051, 1300), 4: (2051, 1300), 8: (9, 1300), 16: (1013, 1300), 32: (1013, 1300)},
    "64 lanes, 16 steps": {1: (5, 2100), 2: (5, 2600), 4: (500, 2600), 8: (500, 2600), 16: (1013, 2600), 32: (1500, 2600)},
}
CASES = [(s, N, *SHAPES[s][N], io, DISCS[(i + j + 2 * k) % 4])
         for j, s in enumerate(SHAPES) for i, N in enumerate(NS) for k, io in enumerate(("f32", "bf16"))]


@pytest.mark.parametrize("shape,N,D,L,io,disc", CASES)
def test_forward_tiles(oracle, shape, N, D, L, io, disc):
    from paper_2602_08810_amd import api
    p = workloads.make_selective(B=1, D=D, N=N, L=L, io=io, gate=N > 1, with_x0=True, seed=N + L, bias=("uniform", -7.0, -6.0))
    y, x, ckpt = api.lrnnx_selective_scan_fwd(**sel_inputs_dev(p, io), disc=disc, return_last_state=True, return_ckpt=True)
    ref = {k: p[k] for k in ("u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "x0")}
    yr, xr = oracle.selective_scan_fwd(disc=disc, **ref)
    last = (L - 1) // 256 * 256                                  # the last checkpoint is the state after that many steps
    cut = {k: (v[..., :last] if k in ("u", "delta", "z") and v is not None else v) for k, v in ref.items()}
    cut["Bm"], cut["Cm"] = ref["Bm"][:, :last], ref["Cm"][:, :last]
    _, cr = oracle.selective_scan_fwd(disc=disc, **cut)
    check_outputs({"y": (host(y), yr, TOL[io]), "x_last": (host(x), xr, 1e-4), "ckpt": (host(ckpt)[:, :, last // 256], cr, 1e-4)}, disc)


# 16 workgroups of channels a launch: 128 chunks, of 2 and of 3 tiles
@pytest.mark.parametrize("N,L,io,disc", [(1, 50001, "f32", "zoh_s6"), (4, 66000, "bf16", "zoh"), (16, 50001, "bf16", "dirac"), (32, 33100, "f32", "bilinear")])
def test_chunks_of_several_tiles(oracle, N, L, io, disc):
    from paper_2602_08810_amd import api
    p = workloads.make_selective(B=16, D=1, N=N, L=L, io=io, gate=True, with_x0=True, seed=N, bias=("uniform", -7.0, -6.0))
    y, x = api.lrnnx_selective_scan_fwd(**sel_inputs_dev(p, io), disc=disc, return_last_state=True, path="chunk_carry")
    yr, xr = oracle.selective_scan_fwd(disc=disc, **{k: p[k] for k in ("u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "x0")})
    check_outputs({"y": (host(y), yr, TOL[io]), "x_last": (host(x), xr, 1e-4)}, disc)


# packed rows enough for 16 lanes (float32: with 16 states or more), several tiles a sequence
@pytest.mark.parametrize("N,io", [(16, "f32"), (32, "f32"), (2, "bf16"), (8, "bf16"), (16, "bf16")])
def test_packed_sixteen_lanes(oracle, N, io):
    import torch
    from paper_2602_08810_amd import api
    lengths = (700, 1, 255, 256, 257, 30, 9, 16)                 # 1524 steps, 190 on average
    p = workloads.make_packed(D=1541, N=N, lengths=lengths, io=io, seed=N)
    t = {k: dev(p[k], io) for k in ("u", "delta", "Bm", "Cm", "z")}
    t.update({k: dev(p[k]) for k in ("A", "Dskip", "delta_bias", "x0")})
    y, x = api.lrnnx_selective_scan_fwd(**t, cu_seqlens=torch.from_numpy(p["cu_seqlens"]).cuda(), return_last_state=True)
    yr, xr = oracle.selective_scan_fwd_packed(cu_seqlens=p["cu_seqlens"], **{k: p[k] for k in ("u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "x0")})
    check_outputs({"y": (host(y), yr, TOL[io]), "x_last": (host(x), xr, 1e-4)})
