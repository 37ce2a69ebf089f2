"""GPU parity of the forward pass where a wavefront takes two states at a time (16 staged states, multipliers e^{Delta A}): each
shape of 64 lanes at the edges of its tile (256, 512, 1024 steps), states alone, and the aggregates of chunks of time."""
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


@pytest.mark.parametrize("N,D,L", [(16, 3, 1), (16, 9, 255), (32, 5, 257), (16, 2101, 65), (16, 2101, 513), (32, 1203, 511),
                                   (16, 5, 1023), (16, 7, 2049), (32, 3, 1025)])
@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("disc", ["zoh_s6", "dirac"])
def test_pairs_of_states(api, oracle, disc, io, N, D, L):
    p = workloads.make_selective(B=1, D=D, N=N, L=L, io=io, gate=L % 2 == 1, with_x0=True, seed=N + L, bias=("uniform", -4.0, -2.0))
    t = sel_inputs_dev(p, io)
    ref = {k: p[k] for k in ("u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "x0")}
    yr, xr, xs = oracle.selective_scan_fwd(disc=disc, return_states=True, **ref)
    before = np.concatenate([p["x0"][:, :, None, :], xs[:, :, 255:L - 1:256, :]], axis=2)     # states entering 0, 256, ...
    for path in ("single_pass", "chunk_carry"):
        y, x, ckpt = api.lrnnx_selective_scan_fwd(**t, disc=disc, path=path, return_last_state=True, return_ckpt=True)
        check_outputs({"y": (host(y), yr, TOL[io]), "x_last": (host(x), xr, 1e-4), "ckpt": (host(ckpt), before, 1e-4)}, path)


@pytest.mark.parametrize("D,L", [(3, 257), (2101, 300), (5, 1025)])
def test_states_alone(api, oracle, D, L):
    """The sweep that the backward pass makes for its checkpoints."""
    p = workloads.make_selective(B=1, D=D, N=16, L=L, io="f32", gate=True, with_x0=True, seed=L, bias=("uniform", -4.0, -2.0))
    t, dy = sel_inputs_dev(p, "f32"), dev(p["dy"], "f32")
    r = oracle.selective_scan_bwd(p["u"], p["delta"], p["A"], p["Bm"], p["Cm"], p["dy"], Dskip=p["Dskip"],
                                  delta_bias=p["delta_bias"], z=p["z"], x0=p["x0"])
    g = api.lrnnx_selective_scan_bwd(**t, dy=dy)
    check_outputs({k: (host(g[k]), r[k], 1e-4) for k in g})
