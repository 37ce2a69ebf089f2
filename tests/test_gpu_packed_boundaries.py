"""GPU parity of packed backward calls whose boundaries do not ascend everywhere: an empty sequence that ends before it starts, first, last and
in the middle, with steps of another sequence before the first boundary, after the last one and outside every sequence between two."""
import numpy as np
import pytest

from paper_2602_08810_amd import workloads
from _util import dev, host, rel_err, sel_inputs_dev

pytestmark = pytest.mark.gpu
TOL_F32 = 1e-4                                              # sums in float32


def poisoned(D, N, L):
    """Outputs full of NaN: whatever a call does not write stays so."""
    import torch
    shapes = dict(du=(D, L), ddelta=(D, L), dz=(D, L), dA=(D, N), dBm=(L, N), dCm=(L, N), dD=(D,), dbias=(D,))
    return {k: torch.full(s, float("nan"), device="cuda") for k, s in shapes.items()}


@pytest.mark.parametrize("workspace", ["own", "none"])     # sums stored and added up by a later launch; added with atomics
@pytest.mark.parametrize("N,D,L,cu,spans", [
    (16, 70, 1200, [0, 900, 500], [(0, 900)]), (8, 300, 3000, [700, 3000, 1], [(700, 3000)]), (4, 33, 900, [800, 100, 700], [(100, 700)]),
    (1, 20, 900, [300, 500, 100, 200], [(300, 500), (100, 200)]), (32, 9, 500, [400, 20], [])])
def test_descending(oracle, N, D, L, cu, spans, workspace):
    import torch
    from paper_2602_08810_amd import api
    p = workloads.make_selective(B=1, D=D, N=N, L=L, io="f32", gate=True, with_dy=True, seed=N + D)
    t = {k: (v if k in ("A", "Dskip", "delta_bias") or v is None else v[0]) for k, v in sel_inputs_dev(p, "f32").items()}
    t.pop("x0", None)
    cud = torch.tensor(cu, dtype=torch.int64, device="cuda")
    _, ckpt = api.lrnnx_selective_scan_fwd(**t, cu_seqlens=cud, return_ckpt=True)
    ws = torch.empty(4 * len(cu), dtype=torch.uint8, device="cuda") if workspace == "none" else None
    g = api.lrnnx_selective_scan_bwd(**t, dy=dev(p["dy"][0], "f32"), ckpt=ckpt, cu_seqlens=cud, outs=poisoned(D, N, L), workspace=ws)
    ref = {k: np.zeros(s) for k, s in dict(du=(D, L), ddelta=(D, L), dz=(D, L), dA=(D, N), dBm=(L, N), dCm=(L, N), dD=D, dbias=D).items()}
    inside = np.zeros(L, dtype=bool)
    for o, e in spans:
        inside[o:e] = True
        r = oracle.selective_scan_bwd_packed(*(p[k][0] for k in ("u", "delta")), p["A"], *(p[k][0] for k in ("Bm", "Cm", "dy")), np.array([o, e]),
                                             Dskip=p["Dskip"], delta_bias=p["delta_bias"], z=p["z"][0])
        for k in ref:
            ref[k] += np.asarray(r[k]).reshape(ref[k].shape)      # (zero outside the sequence)
    for k in ("dA", "dBm", "dCm", "dD", "dbias"):
        assert rel_err(host(g[k]), ref[k]) <= TOL_F32, k
    for k in ("du", "ddelta", "dz"):
        got = host(g[k])
        assert np.isnan(got[:, ~inside]).all(), k                 # steps outside every sequence are not touched
        if spans:
            assert rel_err(got[:, inside], ref[k][:, inside]) <= TOL_F32, k


@pytest.mark.parametrize("N,L,cu", [(16, 70001, [500, 1100, 1300]), (32, 140003, [139000, 139500, 140003]), (1, 150001, [0, 10, 400])])
def test_long_axis_of_few_steps(oracle, N, L, cu):
    """Most of the axis unused: more workgroups clear it, the most there are in the second case."""
    import torch
    from paper_2602_08810_amd import api
    D, o, e = 6, cu[0], cu[-1]
    p = workloads.make_selective(B=1, D=D, N=N, L=e - o, io="f32", gate=True, with_dy=True, seed=N)
    t = {k: (v if k in ("A", "Dskip", "delta_bias") or v is None else v[0]) for k, v in sel_inputs_dev(p, "f32").items()}
    t.pop("x0", None)

    def spread(x, time):                                    # on the long axis, NaN around
        out = torch.full([L if i == time else n for i, n in enumerate(x.shape)], float("nan"), device="cuda")
        out.narrow(time, o, e - o).copy_(x)
        return out
    t = {k: (v if k in ("A", "Dskip", "delta_bias") else spread(v, 0 if k in ("Bm", "Cm") else 1)) for k, v in t.items()}
    g = api.lrnnx_selective_scan_bwd(**t, dy=spread(dev(p["dy"][0], "f32"), 1), cu_seqlens=torch.tensor(cu, device="cuda"), outs=poisoned(D, N, L))
    r = oracle.selective_scan_bwd_packed(*(p[k][0] for k in ("u", "delta")), p["A"], *(p[k][0] for k in ("Bm", "Cm", "dy")), np.array(cu) - o,
                                         Dskip=p["Dskip"], delta_bias=p["delta_bias"], z=p["z"][0])
    for k in ("dBm", "dCm"):
        got, ref = host(g[k]), np.zeros((L, N))
        ref[o:e] = np.asarray(r[k]).reshape(e - o, N)
        assert rel_err(got, ref) <= TOL_F32, k
    for k in ("dA", "dD", "dbias"):
        assert rel_err(host(g[k]), r[k]) <= TOL_F32, k
