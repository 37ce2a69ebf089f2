"""GPU parity of the three ways in which a backward call adds up dA, dD and dbias, by the room in its workspace: partial sums of the batch entries behind
the tile sums of dBm and dCm, tile sums alone, neither.  The workspace and every output are full of NaN before each call, and what a call
left in the workspace shows which way it took.  Also packed complex batches with steps before and after the sequences."""
import ctypes

import numpy as np
import pytest

from paper_2602_08810_amd import workloads
from _util import dev, host, rel_err, sel_inputs_dev

pytestmark = pytest.mark.gpu
TOL_F32 = 1e-4                                              # sums in float32, whatever the type of the inputs
KEYS = ("dA", "dBm", "dCm", "dD", "dbias")


def nan(shape, dtype=None):
    import torch
    return torch.full(shape, complex("nan+nanj") if dtype else float("nan"), dtype=dtype or torch.float32, device="cuda")


def rooms(need, B, D, floats):
    """(tile sums, sums of the entries) in bytes of a call with checkpoints whose size query says `need`, and the rooms to test."""
    entries = 4 * B * D * (floats + 2) if 1 < B <= 32 else 0
    tiles = need - 256 - entries                            # (256: for a workspace that starts anywhere; these start on such a boundary)
    assert tiles > 0 and tiles % (2 * floats * 1024) == 0   # both maps of whole tiles of 256 steps
    full = [("all", need)]
    return tiles, entries, full + ([("tiles", tiles + entries - 4)] if entries else []) + [("neither", tiles - 4)]


def check_use(ws, way, tiles, entries, stored):
    """What of the workspace was written: 0xff bytes everywhere else."""
    used = lambda a, b: bool((ws[a:b] != 0xff).any())
    assert used(0, min(tiles, ws.numel())) == (way != "neither")
    assert used(tiles, tiles + entries) == (way == "all" and stored) if ws.numel() > tiles else True


@pytest.mark.parametrize("B,D,N,L,G,skip", [(1, 37, 16, 300, 1, True), (2, 33, 4, 700, 1, True), (2, 530, 16, 520, 2, False), (32, 5, 8, 257, 1, True),
                                            (33, 5, 8, 257, 1, True), (5, 130, 32, 300, 1, True), (3, 40, 1, 600, 2, False)])
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
    tiles, entries, each = rooms(int(api.lib().lrnnx_selective_scan_bwd_workspace_bytes(ctypes.byref(a))), B, D, N)
    maps = tuple(t["Bm"].shape)
    for way, room in each:
        ws = torch.full((room,), 0xff, dtype=torch.uint8, device="cuda")
        assert ws.data_ptr() % 256 == 0
        outs = dict(dA=nan((D, N)), dBm=nan(maps), dCm=nan(maps), dbias=nan((D,)), du=nan((B, D, L)), **({"dD": nan((D,))} if skip else {}))
        g = api.lrnnx_selective_scan_bwd(**t, dy=dy, ckpt=ckpt, path="single_pass", workspace=ws, outs=outs)
        check_use(ws, way, tiles, entries, stored=entries > 0)
        errs = {k: rel_err(host(g[k]), r[k]) for k in KEYS + ("du",) if r[k] is not None}
        assert "dA" in errs and all(e <= TOL_F32 for e in errs.values()), (way, errs)


@pytest.mark.parametrize("N,D,cu,L", [(16, 70, [3, 300, 300, 901], 1000), (4, 33, [0, 700], 900), (8, 40, [17] + list(range(40, 1040, 31)), 1100),
                                      (8, 40, [17] + list(range(40, 1040, 32)), 1100), (1, 30, [0, 5, 513, 800], 800)])
def test_packed(oracle, N, D, cu, L):
    import torch
    from paper_2602_08810_amd import api
    p = workloads.make_selective(B=1, D=D, N=N, L=L, io="f32", gate=True, with_dy=True, seed=N + D)
    t = {k: (v if k in ("A", "Dskip", "delta_bias") or v is None else v[0]) for k, v in sel_inputs_dev(p, "f32").items()}
    t.pop("x0", None)
    cud = torch.tensor(cu, dtype=torch.int64, device="cuda")
    _, ckpt = api.lrnnx_selective_scan_fwd(**t, cu_seqlens=cud, return_ckpt=True)
    q = {k: p[k][0] for k in ("u", "delta", "Bm", "Cm", "dy", "z")}
    r = oracle.selective_scan_bwd_packed(q["u"], q["delta"], p["A"], q["Bm"], q["Cm"], q["dy"], np.asarray(cu), Dskip=p["Dskip"],
                                         delta_bias=p["delta_bias"], z=q["z"])
    a = api.BwdArgs()
    a.struct_size = ctypes.sizeof(api.BwdArgs)
    a.B, a.D, a.N, a.L, a.cu_seqlens, a.ckpt = len(cu) - 1, D, N, L, 0x1000, 0x1000
    tiles, entries, each = rooms(int(api.lib().lrnnx_selective_scan_bwd_workspace_bytes(ctypes.byref(a))), len(cu) - 1, D, N)
    for way, room in each:
        ws = torch.full((room,), 0xff, dtype=torch.uint8, device="cuda")
        assert ws.data_ptr() % 256 == 0
        outs = dict(dA=nan((D, N)), dBm=nan((L, N)), dCm=nan((L, N)), dD=nan((D,)), dbias=nan((D,)))
        g = api.lrnnx_selective_scan_bwd(**t, dy=dev(q["dy"], "f32"), cu_seqlens=cud, ckpt=ckpt, workspace=ws, outs=outs)
        check_use(ws, way, tiles, entries, stored=entries > 0)
        for k in KEYS:                                      # (dBm and dCm whole: zero outside every sequence)
            got, ref = host(g[k]), np.asarray(r[k])
            assert rel_err(got, ref.reshape(got.shape)) <= TOL_F32, (way, k)


@pytest.mark.parametrize("N,D,cu,L", [(16, 700, [40, 900], 1000), (16, 600, [11, 300, 300, 901, 1400], 1500), (4, 2300, [5, 700, 1030], 1100),
                                      (16, 500, [7] + list(range(30, 1050, 30)), 1090)])
def test_packed_complex_with_unused_steps(oracle, N, D, cu, L):
    """Over the 4 MiB of tile sums from which they go through the workspace: one sequence, several, more than a thread adds up."""
    import torch
    from paper_2602_08810_amd import api
    p = workloads.make_selective_complex(B=1, D=D, N=N, L=L, io="f32", gate=True, seed=N + D)
    dy = np.random.Generator(np.random.PCG64(D)).standard_normal((D, L), dtype=np.float32)
    maps = {k: torch.view_as_complex(torch.from_numpy(np.ascontiguousarray(p[k][0])).cuda()) for k in ("Bm", "Cm")}
    t = dict(u=dev(p["u"][0], "f32"), delta=dev(p["delta"][0], "f32"), A=torch.from_numpy(p["A"]).cuda(), Dskip=dev(p["Dskip"]),
             delta_bias=dev(p["delta_bias"]), z=dev(p["z"][0], "f32"), **maps)
    cud = torch.tensor(cu, dtype=torch.int64, device="cuda")
    _, ckpt = api.lrnnx_selective_scan_fwd_complex(**t, cu_seqlens=cud, return_ckpt=True)
    c = {k: p[k][0, ..., 0].astype(np.float64) + 1j * p[k][0, ..., 1] for k in ("Bm", "Cm")}
    r = oracle.selective_scan_bwd_complex_packed(p["u"][0], p["delta"][0], p["A"], c["Bm"], c["Cm"], dy, np.asarray(cu), Dskip=p["Dskip"],
                                                 delta_bias=p["delta_bias"], z=p["z"][0])
    need = api.lrnnx_workspace_bytes(api.WS_BWD_COMPLEX, len(cu) - 1, D, N, L, api.F32, 1, True)
    for room in (need, 64):                                 # tile sums in the workspace; atomics
        ws = torch.full((room,), 0xff, dtype=torch.uint8, device="cuda")
        c64 = torch.complex64
        outs = dict(dA=nan((D, N), c64), dBm=nan((L, N), c64), dCm=nan((L, N), c64), dD=nan((D,)), dbias=nan((D,)))
        g = api.lrnnx_selective_scan_bwd_complex(**t, dy=dev(dy, "f32"), cu_seqlens=cud, ckpt=ckpt, workspace=ws, outs=outs)
        assert bool((ws[:4 << 20] != 0xff).any()) == (room == need)
        for k in KEYS:
            got, ref = g[k].cpu().numpy(), np.asarray(r[k])
            assert float(np.abs(got - ref.reshape(got.shape)).max() / np.abs(ref).max()) <= TOL_F32, (room, k)      # (NaN fails)
