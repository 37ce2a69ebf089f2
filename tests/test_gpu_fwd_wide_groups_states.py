"""GPU parity of the forward kernels with twelve channels a workgroup at sizes that take them: with checkpoints, without (a plain forward call) and
without outputs (the forward sweep of a backward call without checkpoints).  A last workgroup with one channel and with all but one, grouped
maps, a tile and a half, last tiles of one step, of less than half and of a quarter."""
import numpy as np
import pytest

from paper_2602_08810_amd import workloads
from _util import TOL, check_outputs, dev, host, rel_err, sel_inputs_dev

pytestmark = pytest.mark.gpu
GRAD_TOL_F32 = 1e-4                                         # sums in float32 over many terms, whatever the type of the inputs


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("N,B,D,G,L,disc", [
    (16, 1, 2101, 1, 400, "zoh_s6"), (16, 1, 3071, 1, 512, "zoh_s6"), (16, 3, 771, 1, 1531, "bilinear"), (8, 2, 1090, 2, 900, "zoh"),
    (32, 1, 2053, 1, 511, "dirac"), (8, 1, 3072, 1, 2049, "zoh_s6"), (16, 2, 1309, 1, 1637, "zoh_s6"), (32, 5, 410, 1, 1736, "zoh_s6")])
def test_each_kernel(oracle, io, N, B, D, G, L, disc):
    from paper_2602_08810_amd import api
    p = workloads.make_selective(B=B, D=D, N=N, L=L, io=io, gate=True, with_x0=True, with_dy=True, seed=N + L, bias=("uniform", -4.0, -2.0),
                                 bc_groups=G)
    t = sel_inputs_dev(p, io)
    ref = {k: p[k] for k in ("u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "x0")}
    y, x = api.lrnnx_selective_scan_fwd(**t, disc=disc, return_last_state=True)
    yr, xr, xs = oracle.selective_scan_fwd(disc=disc, return_states=True, **ref)
    check_outputs({"y": (host(y), yr, TOL[io]), "x_last": (host(x), xr, 1e-4)}, disc)
    yc, ckpt = api.lrnnx_selective_scan_fwd(**t, disc=disc, return_ckpt=True)
    before = np.concatenate([p["x0"][:, :, None, :], xs[:, :, 255:L - 1:256, :]], axis=2)
    check_outputs({"y": (host(yc), yr, TOL[io]), "ckpt": (host(ckpt), before, 1e-4)}, disc)
    g = api.lrnnx_selective_scan_bwd(**t, dy=dev(p["dy"], io), disc=disc, want_dx0=True, path="single_pass")
    r = oracle.selective_scan_bwd(dy=p["dy"], disc=disc, delta_softplus=True, **ref)
    tol = {k: TOL[io] if k in ("du", "ddelta", "dz") else GRAD_TOL_F32 for k in g if g[k] is not None and r.get(k) is not None}
    bad = {k: e for k, v in tol.items() for e in [rel_err(host(g[k]), np.asarray(r[k]))] if not e <= v}
    assert {"du", "dz", "dA", "dBm", "dx0"} <= set(tol) and not bad, bad
