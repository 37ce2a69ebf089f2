"""Scans with one workgroup to a block of columns: edges of tiles, of a lane's steps and of column blocks, against float64."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2602_08810_amd import api as _api
    _api.lib()
    return _api


def _shape(api, kind, B, P, L):
    """The column scan's shape that a call takes (lrnnx::column_shape): 0 none, LTI 1: 4 columns x tiles of 1024 steps, 2: 16 x 128, real
    1: 8 x 512, 2: 16 x 128, 3: 32 x 128."""
    if kind == "complex":
        return 0
    return ctypes.CDLL(api.LIB_PATH)._ZN5lrnnx12column_shapeEbiil(kind == "lti", B, P, ctypes.c_int64(L))


def _reference(a, b, x0):
    a, b = a.cpu().numpy(), b.cpu().numpy()
    wide = np.complex128 if np.iscomplexobj(b) else np.float64
    x = np.zeros((b.shape[0], b.shape[2]), wide) if x0 is None else x0.cpu().numpy().astype(wide)
    out = np.empty(b.shape, wide)
    for k in range(b.shape[1]):
        x = (a if a.ndim == 1 else a[:, k]).astype(wide) * x + b[:, k]
        out[:, k] = x
    return out


def _check(api, kind, B, P, L):
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


# around whole tiles and blocks of columns; the longer ones of real coefficients, and complex ones, take the chained scan
@pytest.mark.parametrize("kind", ["lti", "real", "complex"])
@pytest.mark.parametrize("B,P,L", [(1, 1, 1), (2, 3, 7), (1, 4, 8), (3, 5, 9), (2, 15, 127), (1, 16, 128), (2, 17, 129), (8, 208, 92), (5, 31, 511),
                                   (2, 8, 512), (3, 9, 513), (1, 7, 1023), (2, 4, 1024), (1, 6, 1025), (2, 13, 2050), (40, 70, 130),
                                   (8, 1024, 2048), (4, 256, 4096)])
def test_edges(api, kind, B, P, L):
    _check(api, kind, B, P, L)


# three tiles or more in every shape, the last one short, the last block of columns not full
@pytest.mark.parametrize("kind,shape,B,P,L", [("lti", 1, 1, 67, 3075), ("lti", 2, 4, 999, 700), ("real", 1, 1, 1999, 1025), ("real", 1, 2, 2001, 1537),
                                              ("real", 2, 8, 699, 389), ("real", 3, 16, 1009, 300)])
def test_shapes(api, kind, shape, B, P, L):
    assert _shape(api, kind, B, P, L) == shape
    _check(api, kind, B, P, L)


# |coefficient| > 1: the powers over a lane's pieces, a wavefront and a tile grow past float32's range (and double's) where the states, of an
# input that comes late, of a tiny one or of a tiny x0, do not.  A state is one term, rounded at each step (2^-24, three times if complex).
@pytest.mark.parametrize("kind,shape,B,P,L", [("lti", 1, 1, 4, 1000), ("lti", 1, 1, 2, 3000), ("lti", 2, 1, 256, 32), ("lti", 2, 1, 256, 127),
                                              ("lti", 2, 4, 1000, 700), ("real", 1, 1, 64, 700), ("real", 2, 1, 64, 32), ("real", 2, 1, 16, 127),
                                              ("real", 2, 8, 700, 700), ("real", 3, 4, 2000, 1100)])
@pytest.mark.parametrize("coef", [1.05, 1.5, -2.1, 1 + 1j, 17.0, 100.0, 70 - 70j, 1e5, 1e20, 1e38])
def test_growing_states_are_finite_as_long_as_they_are(api, kind, shape, B, P, L, coef):
    if kind == "real":
        coef = abs(coef)
    assert _shape(api, kind, B, P, L) == shape
    dtype = torch.float32 if kind == "real" else torch.complex64
    a = torch.full((P,) if kind == "lti" else (B, L, P), coef, dtype=dtype, device="cuda")
    scan = api.lrnnx_lti_diag_scan if kind == "lti" else api.lrnnx_diag_scan
    grow = np.log(abs(coef))
    for first, value, range_ in ((True, 1e-30, 150), (False, 1.0, 80), (False, 1e-30, 150)):      # x0, late input, tiny late input
        n = min(L - 1, int(range_ / grow))               # steps that the state has up to its largest value
        b, x0 = torch.zeros(B, L, P, dtype=dtype, device="cuda"), None
        if first:
            x0 = torch.full((B, P), value, dtype=dtype, device="cuda")
            a_, b_ = (a if kind == "lti" else a[:, :n].contiguous()), b[:, :n].contiguous()
            if _shape(api, kind, B, P, n) == 0:      # (the chained scan: not what is tested here)
                continue
        else:
            a_, b_ = a, b
            b[:, L - 1 - n] = value
        want = _reference(a_, b_, x0)
        assert np.abs(want).max() < 3e38
        x = scan(a_, b_, x0=x0).cpu().numpy()
        assert (np.abs(x - want) <= 3 * 2.0 ** -24 * (n + 16) * np.abs(want)).all(), (first, value)


# a coefficient of zero ends what came before, however large the products of those after it (beyond double's range from 16 steps on)
@pytest.mark.parametrize("shape,B,P,L", [(1, 1, 64, 700), (2, 1, 64, 32), (2, 1, 16, 127), (2, 8, 700, 700), (3, 4, 2000, 1100)])
@pytest.mark.parametrize("at", [0.0, 0.2, 0.6])
def test_zero_before_large_coefficients(api, shape, B, P, L, at):
    assert _shape(api, "real", B, P, L) == shape
    at = int(at * L)
    a, b = torch.full((B, L, P), 1e20, device="cuda"), torch.zeros(B, L, P, device="cuda")
    a[:, :at], a[:, at] = 0.999, 0.0
    b[:, -1] = 1.0
    x0 = torch.ones(B, P, device="cuda")
    x = api.lrnnx_diag_scan(a, b, x0=x0).cpu().numpy()
    want = _reference(a, b, x0)
    assert (np.abs(x - want) <= 2.0 ** -24 * (at + 16) * np.abs(want)).all()
