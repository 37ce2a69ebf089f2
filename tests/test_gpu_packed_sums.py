"""Sums of dBm and dCm of packed batches around the sizes where four threads share an element: results of each sequence on its own."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# 16-state slots have 8 workgroups and 32-state ones 16: below three halves of the chip, between that and three a CU, beyond it; short last
# tiles and empty sequences
@pytest.mark.parametrize("N,lengths", [
    (16, [2048] * 4), (16, [1900, 0, 2049, 2048, 1, 2047, 2305, 2500]), (16, [2048] * 12), (32, [1023, 1025, 0, 2048, 1000]), (8, [2048] * 14),
    (8, [2000, 0] * 12)])
def test_packed_sums(N, lengths):
    from paper_2602_08810_amd import api
    D, S, L = 640, len(lengths), sum(lengths)
    g = torch.Generator(device="cuda").manual_seed(N * 31 + S)
    r = lambda *s: torch.randn(s, generator=g, device="cuda")
    u, delta, dy, Bm, Cm = r(D, L), r(D, L), r(D, L), r(L, N), r(L, N)
    A, bias = -torch.exp(r(D, N).clamp(-1, 1)), r(D) - 2
    cu = torch.tensor([sum(lengths[:i]) for i in range(S + 1)], device="cuda")
    got = api.lrnnx_selective_scan_bwd(u=u, delta=delta, A=A, Bm=Bm, Cm=Cm, delta_bias=bias, dy=dy, cu_seqlens=cu)
    at = 0
    for n in lengths:
        if n:
            cut = slice(at, at + n)
            rows = {k: v[None, :, cut].contiguous() for k, v in dict(u=u, delta=delta, dy=dy).items()}
            one = api.lrnnx_selective_scan_bwd(**rows, A=A, Bm=Bm[None, cut].contiguous(), Cm=Cm[None, cut].contiguous(), delta_bias=bias, path="single_pass")
            for k in ("dBm", "dCm"):
                # (the bar of all float32 results)
                assert torch.allclose(got[k][cut], one[k][0], rtol=1e-4, atol=1e-4 * float(one[k].abs().max() + 1e-3)), (k, at, n)
        at += n
