"""Packed batches whose workgroups rank the sequences themselves: every sequence is taken once, whatever the lengths, with the
results of a batch of its own."""
import pytest
import torch

import test_gpu_packed
import test_gpu_packed_complex

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2602_08810_amd import api as _api
    _api.lib()
    return _api


def _inputs(cplx, D, L, N, S):
    g = torch.Generator(device="cuda").manual_seed(S * 4099 + D)
    r = lambda *s: torch.randn(s, generator=g, device="cuda")
    A = -torch.exp(r(D, N).clamp(-1, 1))
    Bm, Cm, x0 = r(L, N), r(L, N), r(S, D, N)
    if cplx:
        A, Bm, Cm, x0 = (torch.complex(v, 0.5 * v.roll(1, 0)) for v in (A, Bm, Cm, x0))
    return dict(u=r(D, L), delta=r(D, L), A=A, Bm=Bm, Cm=Cm, Dskip=r(D), delta_bias=r(D) - 2, z=r(D, L), x0=x0), r(D, L)


def _close(a, b):
    a, b = (torch.view_as_real(v) if v.is_complex() else v for v in (a, b))
    return torch.allclose(a, b, rtol=1e-4, atol=1e-4 * float(b.abs().max() + 1e-3))       # (the bar of all float32 results)


# The backward pass (with 4 states the forward pass keeps the caller's order): few workgroups and more than the chip holds; 2, 63 and 64 sequences (one a
# lane), 65 (an order formed by a launch of its own); ties, empty sequences, bounds outside the axis
@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("D,lengths", [
    (40, [300, 20]), (40, [20, 300, 300, 0, 20]), (2600, [100, 17, 300, 300, 0, 64, 1, 257]),
    (640, [(7 * i) % 61 + (200 if i % 9 == 0 else 0) for i in range(63)]), (640, [(5 * i) % 47 for i in range(64)]),
    (640, [(5 * i) % 47 for i in range(65)])], ids=["2", "5", "8", "63", "64", "65"])
def test_every_sequence_once(api, cplx, D, lengths):
    N, S, L = 4, len(lengths), sum(lengths)
    fwd = api.lrnnx_selective_scan_fwd_complex if cplx else api.lrnnx_selective_scan_fwd
    bwd = api.lrnnx_selective_scan_bwd_complex if cplx else api.lrnnx_selective_scan_bwd
    p, dy = _inputs(cplx, D, L, N, S)
    cu = torch.tensor([sum(lengths[:i]) for i in range(S + 1)], device="cuda")
    cu[0], cu[-1] = -5, L + 1000                         # clamped to the axis
    y, last = fwd(**p, cu_seqlens=cu, return_last_state=True)
    g = bwd(**p, dy=dy, cu_seqlens=cu, want_dx0=True)
    at = 0
    for b, n in enumerate(lengths):
        if n == 0:
            assert torch.equal(last[b], p["x0"][b])
            continue
        piece = dict(p, x0=p["x0"][b:b + 1])
        for k in ("Bm", "Cm"):
            piece[k] = p[k][None, at:at + n].contiguous()
        for k in ("u", "delta", "z"):
            piece[k] = p[k][None, :, at:at + n].contiguous()
        y1, last1 = fwd(**piece, return_last_state=True, path="single_pass")
        g1 = bwd(**piece, dy=dy[None, :, at:at + n].contiguous(), want_dx0=True, path="single_pass")
        assert _close(y[:, at:at + n], y1[0]) and _close(last[b], last1[0]) and _close(g["dx0"][b], g1["dx0"][0]), b
        for k in ("du", "ddelta", "dz"):
            assert _close(g[k][:, at:at + n], g1[k][0]), (b, k)
        for k in ("dBm", "dCm"):
            assert _close(g[k][at:at + n], g1[k][0]), (b, k)
        at += n


# The forward pass ranks with 16 lanes a channel, at least 8 states and more workgroups of 16 channels than the chip holds (768): 64 sequences, one
# a lane, and fewer, with ties and empty ones among them; outputs, last states and checkpoints, with the latter read by the backward pass or written by it
@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("io,N", [("f32", 8), ("f32", 16), ("bf16", 8), ("bf16", 16)])
@pytest.mark.parametrize("D,lengths", [(520, [(11 * i) % 61 + (300 if i % 13 == 5 else 0) for i in range(64)]),
                                       (1400, [(29 * i) % 97 + (257 if i % 7 == 6 else 0) for i in range(24)])], ids=["64", "24"])
def test_forward_ranks(api, oracle, cplx, io, N, D, lengths):
    check = (test_gpu_packed_complex if cplx else test_gpu_packed)._check
    check(api, oracle, D, N, lengths, io, seed=N + D, with_ckpt=D == 520)


@pytest.mark.parametrize("cplx", [False, True])
def test_long_axis(api, cplx):
    """Sequences on a time axis of 2^25 steps, from where on a length and an index do not fit one word: the results of a short axis."""
    lengths, at, L = [300, 17, 300, 0, 513, 64], 4099, 1 << 25
    S, N, D = len(lengths), 1, 1
    p, dy = _inputs(cplx, D, sum(lengths), N, S)
    cu = torch.tensor([sum(lengths[:i]) for i in range(S + 1)], device="cuda")
    bwd = api.lrnnx_selective_scan_bwd_complex if cplx else api.lrnnx_selective_scan_bwd
    want = bwd(**p, dy=dy, cu_seqlens=cu, want_dx0=True)
    cut, wide = slice(at, at + sum(lengths)), dict(p)
    for k, v in dict(p, dy=dy).items():
        if k in ("u", "delta", "z", "dy"):
            wide[k] = torch.zeros(D, L, device="cuda")
            wide[k][:, cut] = v
        elif k in ("Bm", "Cm"):
            wide[k] = torch.zeros(L, N, dtype=v.dtype, device="cuda")
            wide[k][cut] = v
    g = bwd(**wide, cu_seqlens=cu + at, want_dx0=True)
    for k, w in want.items():
        got = g[k][:, cut] if k in ("du", "ddelta", "dz") else g[k][cut] if k in ("dBm", "dCm") else g[k]
        assert _close(got, w), k
