"""GPU: loads that go past the caches return what ordinary ones do.  Large forward calls take them from a size on, so two
halves of the batch, each below it, must give the same bits; adjoints take them where every row is whole cache lines, so
the same tensors one element further in memory must.  (An adjoint's stores are non-temporal whatever the rows, but for real values:
there the two calls differ in loads and stores, elsewhere in the loads.)"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    import torch
    assert torch.cuda.is_available()
    from paper_2602_08810_amd import api as _api
    _api.lib()
    return _api


def _rand(shape, cplx, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.complex64 if cplx else torch.float32)


def _shifted(t):
    """The same values, one element further than a cache line's start."""
    import torch
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    buf[1:] = t.reshape(-1)
    return buf[1:].view(t.shape)


# L: just past the size (384 MiB read and written), the last group of steps cut short
@pytest.mark.parametrize("kind,L", [("lti", 3073), ("real", 4099), ("complex", 2050)])
def test_forward_past_the_caches(api, kind, L):
    import torch
    B, P = 8, 1024
    b = _rand((B, L, P), kind != "real", 1)
    if kind == "lti":
        lam = 0.99 * torch.exp(1j * _rand((P,), False, 2))
        scan = lambda s: api.lrnnx_lti_diag_scan(lam, b[s])
    else:
        a = _rand((B, L, P), kind != "real", 3) * 0.4
        scan = lambda s: api.lrnnx_diag_scan(a[s], b[s])
    x = scan(slice(None))
    assert torch.equal(x[:4], scan(slice(0, 4))) and torch.equal(x[4:], scan(slice(4, 8)))


@pytest.mark.parametrize("kind", ["lti", "real", "complex"])
@pytest.mark.parametrize("B,P,L", [(2, 32, 129), (1, 64, 4097), (3, 160, 700), (1, 96, 100)])
def test_adjoint_of_whole_lines(api, kind, B, P, L):
    import torch
    v, gx = (_rand((B, L, P), kind != "real", s) for s in (1, 2))
    assert P * v.element_size() % 128 == 0 and v.data_ptr() % 128 == 0 and gx.data_ptr() % 128 == 0, "whole lines"
    if kind == "lti":
        lam = 0.99 * torch.exp(1j * _rand((P,), False, 3))
        x = api.lrnnx_lti_diag_scan(lam, v)
        got = api.lrnnx_lti_diag_scan_bwd(lam, x, gx)
        ref = api.lrnnx_lti_diag_scan_bwd(lam, _shifted(x), _shifted(gx))
        assert torch.equal(got[0], ref[0]) and torch.equal(got[2], ref[2])
        # dlam is summed with atomics: each sum of B * ceil(L/128) parts in another order
        assert (got[1] - ref[1]).abs().max() <= 1e-5 * ref[1].abs().max()
    else:
        a = _rand((B, L, P), kind != "real", 3) * 0.4
        x = api.lrnnx_diag_scan(a, v)
        got = api.lrnnx_diag_scan_bwd(a, x, gx)
        ref = api.lrnnx_diag_scan_bwd(_shifted(a), _shifted(x), _shifted(gx))
        assert all(torch.equal(g, r) for g, r in zip(got, ref))
