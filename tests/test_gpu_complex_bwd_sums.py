"""GPU parity of the complex backward pass at the edges of its mapping: pieces of 8 steps, tiles of 256, odd channel counts (channels
are walked in pairs), each number of wavefronts per workgroup, and both ways of summing dBm and dCm over workgroups: through
the workspace (calls of some size) and with float atomics (the others, and callers without room for the sums)."""
import numpy as np
import pytest

from paper_2602_08810_amd import workloads
from test_gpu_selective_complex_bwd import _run, api  # noqa: F401  (api: fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("N", [1, 2, 4, 8, 16])
def test_edges_of_pieces_and_tiles(api, oracle, N, io):
    for i, (B, D, L) in enumerate([(1, 3, 7), (2, 5, 9), (1, 2, 255), (1, 33, 257), (2, 1, 513), (1, 9, 1)]):
        _run(api, oracle, B, D, N, L, io, ("zoh_s6", "zoh", "bilinear", "dirac")[(i + N) % 4], gate=i % 2 == 0, x0=i % 3 == 0,
             seed=400 + i, use_ckpt=i % 2 == 1)


# over the line from which the sums go through the workspace (the last: rows of one tile)
@pytest.mark.parametrize("N,D,L,groups", [(1, 2070, 600, 1), (2, 771, 700, 1), (4, 515, 777, 1), (8, 600, 513, 2), (16, 270, 1029, 1),
                                          (1, 6000, 250, 1)])
@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_sums_with_and_without_workspace(api, oracle, io, N, D, L, groups):
    import torch
    g = _run(api, oracle, 2, D, N, L, io, "zoh_s6", gate=True, x0=True, seed=N + L, groups=groups, path="single_pass", use_ckpt=True)
    p = workloads.make_selective_complex(B=2, D=D, N=N, L=L, io=io, gate=True, seed=N + L, with_x0=True, bc_groups=groups)
    from _util import dev
    from test_gpu_selective_complex_bwd import _maps_dev
    t = dict(u=dev(p["u"], io), delta=dev(p["delta"], io), A=torch.from_numpy(p["A"]).cuda(), Bm=_maps_dev(p["Bm"], io),
             Cm=_maps_dev(p["Cm"], io), Dskip=dev(p["Dskip"]), delta_bias=dev(p["delta_bias"]), z=dev(p["z"], io),
             x0=torch.from_numpy(p["x0"]).cuda())
    dy = workloads._io_round(np.random.Generator(np.random.PCG64(N + L + 77)).standard_normal((2, D, L), dtype=np.float32), io)
    _, ckpt = api.lrnnx_selective_scan_fwd_complex(**t, return_ckpt=True)
    call = lambda **kw: api.lrnnx_selective_scan_bwd_complex(**t, dy=dev(dy, io), ckpt=ckpt, path="single_pass", want_dx0=True, **kw)
    again, small = call(), call(workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
    for k in ("du", "ddelta", "dz", "dx0"):
        assert torch.equal(g[k], again[k]) and torch.equal(g[k], small[k]), k
    for k in ("dBm", "dCm"):
        assert torch.equal(g[k], again[k]), k                       # through the workspace: a fixed order
        err = (g[k] - small[k]).abs().max() / g[k].abs().max()
        assert err <= 2e-5, (k, float(err))                         # float32 sums of up to some 10^2 workgroups, in any order
