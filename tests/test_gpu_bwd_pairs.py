"""GPU parity of the backward pass where a wavefront takes two states at a time (N = 16, multipliers e^{Delta A}): the rows of 16
lanes hold alternate pieces of eight steps, so lengths lie around pieces (8), pairs of them (16), rows (128) and tiles (256)."""
import pytest

from paper_2602_08810_amd import workloads
from _util import TOL, check_outputs, dev, host, sel_inputs_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2602_08810_amd import api as _api
    _api.lib()
    return _api


@pytest.mark.parametrize("D,L", [(3, 1), (2, 8), (3, 9), (5, 17), (3, 127), (2, 136), (3, 255), (4, 257), (9, 520)])
@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("disc", ["zoh_s6", "dirac"])
def test_pairs_of_states(api, oracle, disc, io, D, L):
    import torch
    p = workloads.make_selective(B=2, D=D, N=16, L=L, io=io, gate=L % 2 == 1, with_x0=True, seed=L, bias=("uniform", -4.0, -2.0))
    t, dy = sel_inputs_dev(p, io), dev(p["dy"], io)
    _, ckpt = api.lrnnx_selective_scan_fwd(**t, disc=disc, return_ckpt=True)
    r = oracle.selective_scan_bwd(p["u"], p["delta"], p["A"], p["Bm"], p["Cm"], p["dy"], Dskip=p["Dskip"],
                                  delta_bias=p["delta_bias"], z=p["z"], x0=p["x0"], disc=disc)
    for workspace in (None, torch.empty(16, dtype=torch.uint8, device="cuda")):      # sums in scratch, and by atomics
        g = api.lrnnx_selective_scan_bwd(**t, dy=dy, ckpt=ckpt, disc=disc, want_dx0=True, path="single_pass", workspace=workspace)
        check_outputs({k: (host(g[k]), r[k], TOL[io] if k in ("du", "ddelta", "dz") else 1e-4) for k in g}, f"{disc} {D} {L}")
