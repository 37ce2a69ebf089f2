"""GPU parity of the chunked backward pass where the aggregates of the chunks are sums of exponentials (a = e^{Delta A}): chunks of
whole tiles, of a few steps, of less than a lane's eight, and memories that reach across several chunks."""
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
