"""The native half of the Python binding against the general path: the same results for the usual forms of a call, and
nothing taken that the general path checks, converts or refuses."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2602_08810_amd import api as _api
    _api.lib()
    return _api


def _scan(io=torch.float32, groups=1, B=2, D=8, L=300, N=16):
    g = torch.Generator(device="cuda").manual_seed(5)
    r = lambda *s, dt=torch.float32: torch.randn(s, generator=g, device="cuda").to(dt)
    maps = (B, groups, L, N) if groups > 1 else (B, L, N)
    return dict(u=r(B, D, L, dt=io), delta=r(B, D, L, dt=io), A=-torch.exp(r(D, N)), Bm=r(*maps, dt=io), Cm=r(*maps, dt=io),
                Dskip=torch.nn.Parameter(r(D)), delta_bias=r(D) - 3, z=r(B, D, L, dt=io), x0=r(B, D, N))


def _step(io=torch.float32, groups=1, cplx=False, B=3, D=8, N=16):
    g = torch.Generator(device="cuda").manual_seed(6)
    r = lambda *s, dt=torch.float32: torch.randn(s, generator=g, device="cuda").to(dt)
    maps = (B, groups, N) if groups > 1 else (B, N)
    if cplx:
        x, A = torch.view_as_complex(r(B, D, N, 2)), torch.complex(-torch.exp(r(D, N)), r(D, N))
        Bm, Cm = r(*maps, 2, dt=io), r(*maps, 2, dt=io)
        if io == torch.float32:
            Bm, Cm = torch.view_as_complex(Bm), torch.view_as_complex(Cm)
    else:
        x, A, Bm, Cm = r(B, D, N), -torch.exp(r(D, N)), r(*maps, dt=io), r(*maps, dt=io)
    return dict(x=x, u=r(B, D, dt=io), delta=r(B, D, dt=io).t().contiguous().t(), A=A, Bm=Bm, Cm=Cm, Dskip=r(D), delta_bias=r(D) - 3,
                z=r(B, D, dt=io))


def _same(a, b):
    assert type(a) is type(b)
    if isinstance(a, dict):
        assert list(a) == list(b)
        a, b = tuple(a.values()), tuple(b.values())
    if not isinstance(a, tuple):
        a, b = (a,), (b,)
    assert len(a) == len(b)
    for p, q in zip(a, b):
        if p is None:
            assert q is None
            continue
        assert p.shape == q.shape and p.dtype == q.dtype and p.stride() == q.stride() and p.requires_grad == q.requires_grad
        # (gradients of the parameters are float atomics: any order of at most 600 terms)
        p, q = (torch.view_as_real(t) if t.is_complex() else t.float() for t in (p.detach(), q.detach()))
        assert torch.allclose(p, q, rtol=1e-5, atol=1e-5 * float(q.abs().max()))


def _taken(api, f, *args, **kw):
    """The native result, and that the public function and its general path give the same."""
    res = getattr(api._native, f.__name__)(args, kw)
    assert res is not None
    _same(res, f.__wrapped__(*args, **kw))
    _same(f(*args, **kw), res)
    return res


def _complex(p):
    """The same scan with complex A, maps and initial state."""
    q = dict(p, A=torch.complex(p["A"], p["A"].roll(1, 0)), x0=torch.complex(p["x0"], p["x0"].roll(1, 0)))
    for k in ("Bm", "Cm"):
        m = torch.stack([p[k], p[k].roll(1, -1)], -1)
        q[k] = m if m.dtype == torch.bfloat16 else torch.view_as_complex(m)
    return q


@pytest.mark.parametrize("io", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("groups", [1, 4])
@pytest.mark.parametrize("cplx", [False, True])
def test_scan_as_the_general_path(api, io, groups, cplx):
    p = _scan(io, groups)
    fwd, bwd = api.lrnnx_selective_scan_fwd, api.lrnnx_selective_scan_bwd
    if cplx:
        p, fwd, bwd = _complex(p), api.lrnnx_selective_scan_fwd_complex, api.lrnnx_selective_scan_bwd_complex
    bare = dict(x0=None, z=None, Dskip=None, delta_bias=None)
    for opts in (dict(), dict(return_last_state=True, disc="zoh"), dict(return_ckpt=True, path="single_pass"),
                 dict(return_last_state=True, return_ckpt=True, delta_softplus=False, cu_seqlens=None, path="chunk_carry",
                      delta=p["delta"].abs(), delta_bias=None), bare):
        _taken(api, fwd, **{**p, **opts})
    out = torch.empty_like(p["u"])
    assert fwd(**p, out=out) is out
    _same(out, fwd.__wrapped__(**p))
    _taken(api, fwd, *p.values())
    dy = torch.randn_like(p["u"])
    ckpt = fwd(**p, return_ckpt=True)[1]
    for opts in (dict(), dict(ckpt=ckpt, want_dx0=True), dict(disc="bilinear", path="single_pass", workspace=None), {**bare, "max_seqlen": None}):
        _taken(api, bwd, **{**p, "dy": dy, **opts})


@pytest.mark.parametrize("io", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("groups", [1, 2])
@pytest.mark.parametrize("cplx", [False, True])
def test_packed_scan_as_the_general_path(api, io, groups, cplx):
    p = _scan(io, groups, B=1, L=700)
    p = {k: (v[0] if v.dim() > 2 and k != "x0" else v) for k, v in p.items()}
    p["x0"] = torch.cat([p["x0"]] * 3)
    fwd, bwd = api.lrnnx_selective_scan_fwd, api.lrnnx_selective_scan_bwd
    if cplx:
        p, fwd, bwd = _complex(p), api.lrnnx_selective_scan_fwd_complex, api.lrnnx_selective_scan_bwd_complex
    cu = torch.tensor([0, 17, 17, 700], device="cuda")
    if not cplx:
        _taken(api, fwd, **p, cu_seqlens=cu)
    _taken(api, fwd, **p, cu_seqlens=cu, return_last_state=True)
    # (slots between the sequences' checkpoints are not written)
    (y, ckpt), (y2, ck2) = (f(**p, cu_seqlens=cu, return_ckpt=True) for f in (fwd, fwd.__wrapped__))
    _same(y, y2)
    assert ckpt.shape == ck2.shape and ckpt.dtype == ck2.dtype
    dy = torch.randn_like(p["u"])
    for opts in (dict(), dict(max_seqlen=683, want_dx0=True), dict(ckpt=None, path="single_pass")):
        _taken(api, bwd, **{**p, "dy": dy, "cu_seqlens": cu, "ckpt": ckpt, **opts})
    # views of the packed output, and the complex pass's shape without anything beside it, are the general path's
    for kw in (dict(out=torch.empty_like(p["u"])),) + ((dict(),) if cplx else ()):
        assert getattr(api._native, fwd.__name__)((), {**p, "cu_seqlens": cu, **kw}) is None
    for bad in (cu.int(), cu.cpu(), cu[:1], cu[::2]):
        assert getattr(api._native, fwd.__name__)((), {**p, "cu_seqlens": bad, "return_ckpt": True}) is None


@pytest.mark.parametrize("cplx", [False, True])
def test_chained_scans_as_the_general_path(api, cplx):
    g = torch.Generator(device="cuda").manual_seed(7)
    r = lambda *s: torch.view_as_complex(torch.randn((*s, 2), generator=g, device="cuda")) if cplx else torch.randn(s, generator=g, device="cuda")
    a, b, x0 = r(2, 130, 70), r(2, 130, 70), r(2, 70)
    a = a / (1 + a.abs())
    for kw in (dict(), dict(x0=x0), dict(x0=x0, return_last_state=True)):
        _taken(api, api.lrnnx_diag_scan, a, b, **kw)
    out = torch.empty_like(b)
    assert api.lrnnx_diag_scan(a, b, out=out) is out
    for kw in (dict(), dict(x0=x0), dict(want_dx0=False)):
        _taken(api, api.lrnnx_diag_scan_bwd, a, out, b, **kw)
    for f, args in ((api.lrnnx_diag_scan, (a, b[:1])), (api.lrnnx_diag_scan, (a.to(torch.complex128), b)), (api.lrnnx_diag_scan_bwd, (a, out, b.transpose(0, 1)))):
        assert getattr(api._native, f.__name__)(args, {}) is None
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    assert api._native.lrnnx_diag_scan((a, b), dict(chain_status=status)) is None
    if not cplx:
        assert api._native.lrnnx_lti_diag_scan((a[0, 0], b), {}) is None
        return
    lam = a[0, 0].contiguous()
    for kw in (dict(), dict(x0=x0, path="chunk_carry"), dict(x0=x0, return_last_state=True), dict(out=torch.empty_like(b))):
        _taken(api, api.lrnnx_lti_diag_scan, lam, b, **kw)
    x = api.lrnnx_lti_diag_scan(lam, b)
    for kw in (dict(), dict(x0=x0), dict(want_dx0=False), dict(out=torch.empty_like(b))):
        _taken(api, api.lrnnx_lti_diag_scan_bwd, lam, x, b, **kw)
    assert api._native.lrnnx_lti_diag_scan((lam, b.conj()), {}) is None
    assert api._native.lrnnx_lti_diag_scan((lam[:3], b), {}) is None


@pytest.mark.parametrize("io", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("groups", [1, 2])
@pytest.mark.parametrize("cplx", [False, True])
def test_step_as_the_general_path(api, io, groups, cplx):
    step = api.lrnnx_selective_step_complex if cplx else api.lrnnx_selective_step
    native = getattr(api._native, step.__name__)
    out = torch.empty(8, 3, dtype=io, device="cuda").t()
    for opts in (dict(), dict(disc="dirac", delta_softplus=False), dict(z=None, Dskip=None, delta_bias=None), dict(out=out)):
        p = {**_step(io, groups, cplx), **opts}
        a, b, c = ({**p, "x": p["x"].clone()} for _ in range(3))
        assert native((), a) is not None
        ya = a["x"]
        yb, yc = step(**b), step.__wrapped__(**{**c, **({"out": out.clone()} if "out" in opts else {})})
        assert yb is out if "out" in opts else True
        assert torch.equal(ya, b["x"]) and torch.equal(b["x"], c["x"]) and torch.equal(yb, yc)


def _unusual():
    """(calls that only the general path takes, or refuses; whether it refuses)"""
    p = _scan()
    t = lambda k, f: {**p, k: f(p[k])}
    yield "rows in another order", t("u", lambda v: v.transpose(0, 1).contiguous().transpose(0, 1)), False
    yield "a broadcast row", t("z", lambda v: v[:, :1].expand(-1, 8, -1)), False
    yield "a mode by number", {**p, "disc": 0}, False
    yield "a truth value that is none", {**p, "delta_softplus": 1}, False
    yield "scratch of the caller's", {**p, "workspace": torch.empty(1 << 16, dtype=torch.uint8, device="cuda")}, False
    yield "a type of its own", t("u", lambda v: v.as_subclass(type("T", (torch.Tensor,), {}))), False
    yield "another type", t("delta", lambda v: v.bfloat16()), True
    yield "maps of another type", t("Bm", lambda v: v.bfloat16()), True
    yield "on the host", t("A", lambda v: v.cpu()), True
    yield "half the channels", t("z", lambda v: v[:, :4]), True
    yield "an unknown mode", {**p, "disc": "euler"}, True
    yield "an unknown argument", {**p, "gate": True}, True
    yield "no A", {k: v for k, v in p.items() if k != "A"}, True
    yield "groups that do not divide", t("Bm", lambda v: torch.stack([v] * 3, 1)) | {"Cm": torch.stack([p["Cm"]] * 3, 1)}, True
    yield "five states", {k: (v[..., :5].contiguous() if k in ("A", "Bm", "Cm", "x0") else v) for k, v in p.items()}, True


def test_unusual_calls_go_the_general_way(api):
    fwd, native = api.lrnnx_selective_scan_fwd, api._native.lrnnx_selective_scan_fwd
    for what, kw, refused in _unusual():
        if what != "five states":                        # (a usual form: the library itself refuses it)
            assert native((), kw) is None, what
        if not refused:
            _same(fwd(**kw), fwd.__wrapped__(**kw))
            continue
        said = []
        for f in (fwd, fwd.__wrapped__):
            with pytest.raises(Exception) as e:
                f(**kw)
            said.append((type(e.value), str(e.value)))
        assert said[0] == said[1], what
    p = _scan()
    assert native((p["u"],), p) is None                  # given twice
    with torch.device("cuda"):                           # a mode that takes over functions
        assert native((), p) is None
    got = []
    torch.func.vmap(lambda v: (got.append(native((), {**p, "u": v})), v)[1])(p["u"].unsqueeze(0))
    assert got == [None]
