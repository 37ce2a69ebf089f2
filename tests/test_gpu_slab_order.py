"""GPU parity of the scans whose workgroups take slabs of 64 columns, where the slabs are dealt to the dies: rows that are not whole cache lines
and numbers of slabs around multiples of eight, many slabs of whole lines, and rows of 8-byte values past the caches."""
import numpy as np
import pytest

from paper_2602_08810_amd import workloads
from _util import rel_err

pytestmark = pytest.mark.gpu


def _err(got, ref):
    got = got.cpu().numpy()
    return max(rel_err(got.real, ref.real), rel_err(got.imag, ref.imag)) if np.iscomplexobj(ref) else rel_err(got, ref)


# slabs: 3, 8, 9, 15, 36, 64 of whole lines; the last two with non-temporal loads of broken lines
@pytest.mark.parametrize("kind,B,P,L", [(k, *s) for k in ("lti", "real", "complex") for s in [
    (1, 130, 513), (2, 250, 260), (3, 129, 700), (5, 161, 300), (9, 199, 257), (16, 256, 300)]] + [("lti", 5, 1237, 4100), ("complex", 5, 1001, 3500)])
def test_slab_order(oracle, kind, B, P, L):
    import torch
    from paper_2602_08810_amd import api
    make = workloads.make_lti if kind == "lti" else workloads.make_diag
    q = make(B=B, P=P, L=L, seed=B + P, with_x0=True, with_gx=True, **({} if kind == "lti" else {"cplx": kind == "complex"}))
    t = {k: torch.from_numpy(q[k]).cuda() for k in q if isinstance(q[k], np.ndarray)}
    if kind == "lti":
        x = api.lrnnx_lti_diag_scan(t["lam"], t["v"], x0=t["x0"])
        got = (x, *api.lrnnx_lti_diag_scan_bwd(t["lam"], x, t["gx"], x0=t["x0"]))
        ref = (oracle.lti_diag_scan(q["lam"], q["v"], x0=q["x0"]), *oracle.lti_diag_scan_bwd(q["lam"], q["v"], q["gx"], x0=q["x0"]))
    else:
        x = api.lrnnx_diag_scan(t["a"], t["b"], x0=t["x0"])
        got = (x, *api.lrnnx_diag_scan_bwd(t["a"], x, t["gx"], x0=t["x0"]))
        ref = (oracle.diag_scan(q["a"], q["b"], x0=q["x0"]), *oracle.diag_scan_bwd(q["a"], q["b"], q["gx"], x0=q["x0"]))
    errs = [_err(g, r) for g, r in zip(got, ref)]
    assert len(errs) == 4 and all(e <= 1e-4 for e in errs), errs
