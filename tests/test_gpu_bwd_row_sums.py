"""GPU parity of dA, dD and dbias where the workgroups of a backward call store their sums and a later launch adds up the batch entries: one
entry, two, as many as a thread adds up and one more; with room for them in the workspace and, a word short, with atomics; real and complex."""
import ctypes

import numpy as np
import pytest

from paper_2602_08810_amd import workloads
from _util import dev, host, rel_err, sel_inputs_dev

pytestmark = pytest.mark.gpu
TOL_F32 = 1e-4                                              # sums in float32, whatever the type of the inputs


@pytest.mark.parametrize("B,D,N,L,G,skip", [(1, 37, 16, 300, 1, True), (2, 33, 4, 700, 1, True), (2, 1030, 16, 520, 2, False),
                                            (32, 5, 8, 257, 1, True), (33, 5, 8, 257, 1, True), (5, 130, 32, 300, 1, True), (3, 40, 1, 600, 2, False)])
def test_real(oracle, B, D, N, L, G, skip):
    import torch
    from paper_2602_08810_amd import api
    p = workloads.make_selective(B=B, D=D, N=N, L=L, io="f32", gate=True, with_dy=True, seed=B + D, bc_groups=G)
    if not skip:
        p["Dskip"] = None
    t, dy = sel_inputs_dev(p, "f32"), dev(p["dy"], "f32")
    _, ckpt = api.lrnnx_selective_scan_fwd(**t, return_ckpt=True)
    r = oracle.selective_scan_bwd(p["u"], p["delta"], p["A"], p["Bm"], p["Cm"], p["dy"], Dskip=p["Dskip"], delta_bias=p["delta_bias"], z=p["z"])
    a = api.BwdArgs()
    a.struct_size = ctypes.sizeof(api.BwdArgs)
    a.B, a.D, a.N, a.L, a.bc_groups, a.path, a.ckpt = B, D, N, L, G, api.PATH["single_pass"], 0x1000
    need = int(api.lib().lrnnx_selective_scan_bwd_workspace_bytes(ctypes.byref(a)))
    for room in (need, need - 4):
        ws = torch.full((room,), 0xff, dtype=torch.uint8, device="cuda")       # (NaN in whatever is read before it is written)
        g = [api.lrnnx_selective_scan_bwd(**t, dy=dy, ckpt=ckpt, path="single_pass", workspace=ws) for _ in range(2)]
        errs = {k: rel_err(host(g[0][k]), r[k]) for k in ("dA", "dBm", "dCm", "dD", "dbias", "du") if r[k] is not None}
        assert "dA" in errs and all(e <= TOL_F32 for e in errs.values()), (room, errs)
        if room == need and B <= 32:                        # always the same order (dD and dbias meet in LDS within a workgroup, in any)
            assert torch.equal(g[0]["dA"], g[1]["dA"])


@pytest.mark.parametrize("B,D,N,L", [(1, 700, 16, 600), (2, 900, 8, 1030), (3, 1200, 2, 700)])
def test_complex(oracle, B, D, N, L):
    import torch
    from paper_2602_08810_amd import api
    p = workloads.make_selective_complex(B=B, D=D, N=N, L=L, io="f32", gate=True, seed=B + D)
    rng = np.random.Generator(np.random.PCG64(D))
    dy = rng.standard_normal((B, D, L), dtype=np.float32)
    maps = {k: torch.view_as_complex(torch.from_numpy(np.ascontiguousarray(p[k])).cuda()) for k in ("Bm", "Cm")}
    t = dict(u=dev(p["u"], "f32"), delta=dev(p["delta"], "f32"), A=torch.from_numpy(p["A"]).cuda(), Dskip=dev(p["Dskip"]),
             delta_bias=dev(p["delta_bias"]), z=dev(p["z"], "f32"), **maps)
    _, ckpt = api.lrnnx_selective_scan_fwd_complex(**t, return_ckpt=True)
    g = api.lrnnx_selective_scan_bwd_complex(**t, dy=dev(dy, "f32"), ckpt=ckpt, path="single_pass")
    c = {k: p[k][..., 0].astype(np.float64) + 1j * p[k][..., 1] for k in ("Bm", "Cm")}
    r = oracle.selective_scan_bwd_complex(p["u"], p["delta"], p["A"], c["Bm"], c["Cm"], dy, Dskip=p["Dskip"], delta_bias=p["delta_bias"], z=p["z"])
    for k in ("dA", "dD", "dbias", "dBm"):
        got, ref = np.asarray(host(g[k]) if not g[k].is_complex() else g[k].cpu().numpy()), np.asarray(r[k])
        assert float(np.abs(got - ref).max() / np.abs(ref).max()) <= TOL_F32, k


@pytest.mark.parametrize("N,D,cu,L", [(16, 70, [3, 300, 300, 901], 1000), (4, 33, [0, 700], 900), (8, 40, [17] + list(range(40, 1040, 31)), 1100),
                                      (1, 30, [0, 5, 513, 800], 800)])
def test_packed(oracle, N, D, cu, L):
    """Also the rows of dBm and dCm outside every sequence, which the same launch clears."""
    import torch
    from paper_2602_08810_amd import api
    p = workloads.make_selective(B=1, D=D, N=N, L=L, io="f32", gate=True, with_dy=True, seed=N + D)
    t = {k: (v if k in ("A", "Dskip", "delta_bias") or v is None else v[0]) for k, v in sel_inputs_dev(p, "f32").items()}
    cud = torch.tensor(cu, dtype=torch.int64, device="cuda")
    t.pop("x0", None)
    q = {k: p[k][0] for k in ("u", "delta", "Bm", "Cm", "dy", "z")}
    r = oracle.selective_scan_bwd_packed(q["u"], q["delta"], p["A"], q["Bm"], q["Cm"], q["dy"], np.asarray(cu), Dskip=p["Dskip"],
                                         delta_bias=p["delta_bias"], z=q["z"])
    a = api.BwdArgs()
    a.struct_size = ctypes.sizeof(api.BwdArgs)
    a.B, a.D, a.N, a.L, a.cu_seqlens = len(cu) - 1, D, N, L, 0x1000
    need = int(api.lib().lrnnx_selective_scan_bwd_workspace_bytes(ctypes.byref(a)))
    inside = np.zeros(L, dtype=bool)
    inside[cu[0]:cu[-1]] = True
    for room in (need, need - 4):
        ws = torch.full((room,), 0xff, dtype=torch.uint8, device="cuda")
        g = api.lrnnx_selective_scan_bwd(**t, dy=dev(q["dy"], "f32"), cu_seqlens=cud, workspace=ws)
        for k in ("dA", "dBm", "dCm", "dD", "dbias"):
            assert rel_err(host(g[k]), r[k]) <= TOL_F32, (room, k)
        assert not host(g["dBm"])[~inside].any() and not host(g["dCm"])[~inside].any()
