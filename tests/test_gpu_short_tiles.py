"""GPU parity where a sequence's last tile is short: its wavefronts take fewer steps a lane (backward 4 up to 128 steps and 2 up to
64, forward with 16 lanes a channel 8 and 4), so lengths lie around 64 and 128 past whole tiles of 256, and around a lane's steps."""
import pytest

from paper_2602_08810_amd import workloads
from _util import TOL, check_outputs, dev, host, sel_inputs_dev

pytestmark = pytest.mark.gpu

DISCS = ["zoh_s6", "zoh", "bilinear", "dirac"]
NAMES = ("u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "x0")


@pytest.fixture(scope="module")
def api():
    from paper_2602_08810_amd import api as _api
    _api.lib()
    return _api


@pytest.mark.parametrize("L", [2, 3, 63, 64, 65, 127, 128, 129, 256 + 64, 256 + 65, 512 + 128, 512 + 129])
@pytest.mark.parametrize("N", [4, 8, 16, 32])
@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_backward(api, oracle, io, N, L):
    import torch
    disc = DISCS[(N // 8 + L) % 4]
    p = workloads.make_selective(B=2, D=5, N=N, L=L, io=io, gate=L % 2 == 1, with_x0=True, seed=N + L, bias=("uniform", -4.0, -2.0))
    t, dy = sel_inputs_dev(p, io), dev(p["dy"], io)
    r = oracle.selective_scan_bwd(dy=p["dy"], disc=disc, **{k: p[k] for k in NAMES})
    _, ckpt = api.lrnnx_selective_scan_fwd(**t, disc=disc, return_ckpt=True)
    for workspace in (None, torch.empty(16, dtype=torch.uint8, device="cuda")):      # sums in scratch, and by atomics
        g = api.lrnnx_selective_scan_bwd(**t, dy=dy, ckpt=ckpt, disc=disc, want_dx0=True, path="single_pass", workspace=workspace)
        check_outputs({k: (host(g[k]), r[k], TOL[io] if k in ("du", "ddelta", "dz") else 1e-4) for k in g}, f"{disc} {N} {L}")


# the chunked path takes 16 lanes a channel; its last chunk ends in the short tile
@pytest.mark.parametrize("L", [256 + 1, 256 + 64, 256 + 65, 512 + 127, 512 + 128, 512 + 129])
@pytest.mark.parametrize("N", [1, 2, 4, 8, 16, 32])
@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_forward(api, oracle, io, N, L):
    disc = DISCS[(N // 4 + L) % 4]
    p = workloads.make_selective(B=2, D=21, N=N, L=L, io=io, gate=True, with_x0=True, seed=N + L, bias=("uniform", -4.0, -2.0))
    y, x, ckpt = api.lrnnx_selective_scan_fwd(**sel_inputs_dev(p, io), disc=disc, return_last_state=True, return_ckpt=True, path="chunk_carry")
    yr, xr, xs = oracle.selective_scan_fwd(disc=disc, return_states=True, **{k: p[k] for k in NAMES})
    check_outputs({"y": (host(y), yr, TOL[io]), "x_last": (host(x), xr, 1e-4), "ckpt": (host(ckpt)[:, :, 1:], xs[:, :, 255:L - 1:256, :], 1e-4)}, disc)


# many rows of short sequences, without vector access (rows that start at odd elements) and with it; states alone too
@pytest.mark.parametrize("L", [33, 64, 65, 128, 129])
@pytest.mark.parametrize("io,N", [("f32", 1), ("bf16", 4), ("bf16", 16)])
def test_many_short_rows(api, oracle, io, N, L):
    import torch
    B, D = 4, 4100
    p = workloads.make_selective(B=B, D=D, N=N, L=L, io=io, gate=True, with_x0=True, seed=N + L, bias=("uniform", -4.0, -2.0))
    t, dy = sel_inputs_dev(p, io), dev(p["dy"], io)
    yr, xr = oracle.selective_scan_fwd(**{k: p[k] for k in NAMES})
    r = oracle.selective_scan_bwd(dy=p["dy"], **{k: p[k] for k in NAMES})
    y, x = api.lrnnx_selective_scan_fwd(**t, return_last_state=True)
    check_outputs({"y": (host(y), yr, TOL[io]), "x_last": (host(x), xr, 1e-4)})
    g = api.lrnnx_selective_scan_bwd(**t, dy=dy, want_dx0=True)
    check_outputs({k: (host(g[k]), r[k], TOL[io] if k in ("du", "ddelta", "dz") else 1e-4) for k in g})
    cu = torch.arange(0, B + 1, device="cuda") * L                                   # the same rows as a packed batch
    flat = {k: t[k].transpose(0, 1).reshape(D, B * L).contiguous() for k in ("u", "delta", "z")}
    maps = {k: t[k].reshape(B * L, N) for k in ("Bm", "Cm")}
    yp, xp = api.lrnnx_selective_scan_fwd(**flat, **maps, **{k: t[k] for k in ("A", "Dskip", "delta_bias", "x0")}, cu_seqlens=cu, return_last_state=True)
    check_outputs({"y": (host(yp.reshape(D, B, L).transpose(0, 1)), yr, TOL[io]), "x_last": (host(xp), xr, 1e-4)})
