"""Scans with one workgroup to a block of columns: edges of tiles, of a lane's steps and of column blocks, against float64."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2602_08810_amd import api as _api
    _api.lib()
    return _api


def _reference(a, b, x0):
    a, b = a.cpu().numpy(), b.cpu().numpy()
    wide = np.complex128 if np.iscomplexobj(b) else np.float64
    x = np.zeros((b.shape[0], b.shape[2]), wide) if x0 is None else x0.cpu().numpy().astype(wide)
    out = np.empty(b.shape, wide)
    for k in range(b.shape[1]):
        x = (a if a.ndim == 1 else a[:, k]).astype(wide) * x + b[:, k]
        out[:, k] = x
    return out


# columns of a workgroup x steps of its tile: LTI 4 x 1024 and 16 x 128, real 8 x 512, 16 x 128 and 32 x 128 (complex: the chained scan)
@pytest.mark.parametrize("kind", ["lti", "real", "complex"])
@pytest.mark.parametrize("B,P,L", [(1, 1, 1), (2, 3, 7), (1, 4, 8), (3, 5, 9), (2, 15, 127), (1, 16, 128), (2, 17, 129), (8, 208, 92), (5, 31, 511),
                                   (2, 8, 512), (3, 9, 513), (1, 7, 1023), (2, 4, 1024), (1, 6, 1025), (2, 13, 2050), (40, 70, 130),
                                   (8, 1024, 2048), (4, 256, 4096)])
def test_edges(api, kind, B, P, L):
    g = torch.Generator(device="cuda").manual_seed(B * 1000003 + P * 1009 + L)
    rand = lambda *s: torch.rand(s, generator=g, device="cuda")
    randn = lambda *s: torch.randn(s, generator=g, device="cuda")
    number = (lambda *s: randn(*s)) if kind == "real" else (lambda *s: torch.view_as_complex(randn(*s, 2)))
    coef = (lambda *s: rand(*s)) if kind == "real" else (lambda *s: torch.polar(0.9 + 0.099 * rand(*s), 6.28 * rand(*s)))
    a, b = coef(P) if kind == "lti" else coef(B, L, P), number(B, L, P)
    scan = api.lrnnx_lti_diag_scan if kind == "lti" else api.lrnnx_diag_scan
    for x0 in (None, number(B, P)):
        want = _reference(a, b, x0)
        x, last = scan(a, b, x0=x0, return_last_state=True)
        # a state is a sum of terms that decay with a memory of at most 1000 steps, each rounded to 2^-24
        for got, ref in ((x, want), (last, want[:, -1])):
            assert np.abs(got.cpu().numpy() - ref).max() <= 3e-5 * np.abs(want).max()
        own = b.clone()
        assert scan(a, own, x0=x0, out=own) is own       # in place
        assert torch.equal(own, x)


def test_growing_states_stay_finite_as_long_as_they_are(api):
    """|lambda| > 1 and inputs that start late: powers over more steps than a wavefront's must not be formed."""
    lam = torch.full((4,), 1.05, dtype=torch.complex64, device="cuda")
    v = torch.zeros(1, 1024, 4, dtype=torch.complex64, device="cuda")
    v[:, 600] = 1.0
    x = api.lrnnx_lti_diag_scan(lam, v)
    want = _reference(lam, v, None)
    assert torch.isfinite(torch.view_as_real(x)).all()
    assert np.abs(x.cpu().numpy() - want).max() <= 1e-4 * np.abs(want).max()
