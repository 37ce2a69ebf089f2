"""GPU parity of the chunked backward pass where the aggregates of the chunks are sums of exponentials (a = e^{Delta A}): chunks of
whole tiles, of a few steps, of less than a lane's eight, of several tiles, and memories that reach across several chunks."""
import numpy as np
import pytest

from paper_2602_08810_amd import workloads
from _util import TOL, check_outputs, dev, host, sel_inputs_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2602_08810_amd import api as _api
    _api.lib()
    return _api


@pytest.mark.parametrize("D,L", [(3, 257), (9, 263), (8, 264), (2, 777), (3, 1025), (5, 2055)])
@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("N,disc", [(1, "dirac"), (2, "zoh"), (4, "zoh_s6"), (8, "zoh"), (16, "zoh_s6"), (16, "bilinear"), (32, "zoh_s6")])
def test_chunks(api, oracle, N, disc, io, D, L):
    p = workloads.make_selective(B=2, D=D, N=N, L=L, io=io, gate=L % 2 == 1, with_x0=True, seed=L + N, bias=("uniform", -7.0, -3.0))
    t, dy = sel_inputs_dev(p, io), dev(p["dy"], io)
    _, ckpt = api.lrnnx_selective_scan_fwd(**t, disc=disc, return_ckpt=True)
    r = oracle.selective_scan_bwd(p["u"], p["delta"], p["A"], p["Bm"], p["Cm"], p["dy"], Dskip=p["Dskip"],
                                  delta_bias=p["delta_bias"], z=p["z"], x0=p["x0"], disc=disc)
    g = api.lrnnx_selective_scan_bwd(**t, dy=dy, ckpt=ckpt, disc=disc, want_dx0=True, path="chunk_carry")
    check_outputs({k: (host(g[k]), r[k], TOL[io] if k in ("du", "ddelta", "dz") else 1e-4) for k in g}, f"{disc} {N} {D} {L}")


# The last chunk of a packed sequence takes whatever the hint leaves over: here one tile of 256 steps a chunk is planned, and the
# kernel's own tiles (512 steps) run to three, the last of 1, 7, 8, 9 and 511 steps.  Memories of thousands of steps reach across
# all of them; 11 channels leave five of a workgroup's wavefronts without one.
@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("N,disc", [(1, "zoh_s6"), (2, "zoh"), (4, "dirac"), (8, "zoh_s6"), (16, "zoh"), (16, "bilinear"), (32, "zoh_s6")])
def test_chunks_of_several_tiles(api, oracle, N, disc, io):
    import torch
    D, hint = 11, 512
    lengths = [256 + n for n in (1024 + 1, 512 + 7, 1024 + 8, 512 + 9, 512 + 511, 5)]
    assert api.lib().lrnnx_selective_scan_bwd_chunks(len(lengths), D, N, hint, 1, 2, 0) == hint // 256
    p = workloads.make_packed(D=D, N=N, lengths=lengths, io=io, seed=N, gap=3)
    p["delta_bias"] = np.random.Generator(np.random.PCG64(N)).uniform(-9.0, -7.0, D).astype(np.float32)
    t, dy, cu = sel_inputs_dev(p, io), dev(p["dy"], io), torch.from_numpy(p["cu_seqlens"]).cuda()
    _, ckpt = api.lrnnx_selective_scan_fwd(**t, disc=disc, cu_seqlens=cu, return_ckpt=True)
    outs = {k: torch.zeros_like(t["u"]) for k in ("du", "ddelta", "dz")}             # (steps outside every sequence are not written)
    g = api.lrnnx_selective_scan_bwd(**t, dy=dy, ckpt=ckpt, disc=disc, cu_seqlens=cu, want_dx0=True, path="chunk_carry",
                                     max_seqlen=hint, outs=outs)
    r = oracle.selective_scan_bwd_packed(p["u"], p["delta"], p["A"], p["Bm"], p["Cm"], p["dy"], p["cu_seqlens"], Dskip=p["Dskip"],
                                         delta_bias=p["delta_bias"], z=p["z"], x0=p["x0"], disc=disc)
    check_outputs({k: (host(g[k]), r[k], TOL[io] if k in ("du", "ddelta", "dz") else 1e-4) for k in g}, f"{disc} {N}")
