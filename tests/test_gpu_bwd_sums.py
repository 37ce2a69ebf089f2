"""GPU parity of the two ways the backward pass sums dBm and dCm over workgroups: partial sums in the workspace added by a
second launch (the binding's default), and float atomics when the caller's workspace has no room for them."""
import numpy as np
import pytest

from paper_2602_08810_amd import workloads
from _util import check_outputs, dev, host, sel_inputs_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2602_08810_amd import api as _api
    _api.lib()
    return _api


# state sizes of each number of wavefronts per workgroup; lengths at the edges of a lane (8), a piece of the second
# launch (256 * 4 / N steps) and a tile (256); odd channel counts (channels are walked in pairs)
@pytest.mark.parametrize("N,D,L", [(1, 5, 257), (2, 3, 255), (4, 9, 513), (8, 17, 129), (16, 11, 65), (16, 40, 300), (32, 7, 289)])
@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_sums_with_and_without_workspace(api, oracle, io, N, D, L):
    import torch
    p = workloads.make_selective(B=2, D=D, N=N, L=L, io=io, gate=True, with_x0=True, seed=N + L, bias=("uniform", -4.0, -2.0))
    t, dy = sel_inputs_dev(p, io), dev(p["dy"], io)
    _, ckpt = api.lrnnx_selective_scan_fwd(**t, return_ckpt=True)
    r = oracle.selective_scan_bwd(p["u"], p["delta"], p["A"], p["Bm"], p["Cm"], p["dy"], Dskip=p["Dskip"],
                                  delta_bias=p["delta_bias"], z=p["z"], x0=p["x0"])
    small = torch.empty(16, dtype=torch.uint8, device="cuda")
    with_sums = api.lrnnx_selective_scan_bwd(**t, dy=dy, ckpt=ckpt, path="single_pass")
    atomics = api.lrnnx_selective_scan_bwd(**t, dy=dy, ckpt=ckpt, path="single_pass", workspace=small)
    for g, where in ((with_sums, "workspace"), (atomics, "atomics")):
        check_outputs({k: (host(g[k]), r[k], 1e-4) for k in ("dBm", "dCm", "dA", "dD", "dbias")}, where)
    assert torch.equal(with_sums["du"], atomics["du"])
    again = api.lrnnx_selective_scan_bwd(**t, dy=dy, ckpt=ckpt, path="single_pass")
    assert torch.equal(with_sums["dBm"], again["dBm"]) and torch.equal(with_sums["dCm"], again["dCm"])   # fixed order
