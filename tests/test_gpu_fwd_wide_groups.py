"""GPU parity of the forward pass with twelve channels a workgroup: the first and last row counts that take it, a last workgroup with one channel
and with all but one, grouped maps, tiles that end early."""
import numpy as np
import pytest

from paper_2602_08810_amd import workloads
from _util import TOL, check_outputs, host, sel_inputs_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("N,B,D,G,L,disc", [
    (16, 1, 2049, 1, 300, "zoh_s6"), (16, 1, 3071, 1, 513, "zoh_s6"), (16, 3, 771, 1, 515, "bilinear"), (8, 2, 1030, 2, 1025, "zoh"),
    (32, 1, 2053, 1, 511, "dirac"), (8, 1, 3072, 1, 9, "zoh_s6")])
def test_forward_wide_groups(oracle, io, N, B, D, G, L, disc):
    from paper_2602_08810_amd import api
    p = workloads.make_selective(B=B, D=D, N=N, L=L, io=io, gate=True, with_x0=True, seed=N + L, bias=("uniform", -4.0, -2.0), bc_groups=G)
    y, x, ckpt = api.lrnnx_selective_scan_fwd(**sel_inputs_dev(p, io), disc=disc, return_last_state=True, return_ckpt=True)
    ref = {k: p[k] for k in ("u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "x0")}
    yr, xr, xs = oracle.selective_scan_fwd(disc=disc, return_states=True, **ref)
    before = np.concatenate([p["x0"][:, :, None, :], xs[:, :, 255:L - 1:256, :]], axis=2)
    check_outputs({"y": (host(y), yr, TOL[io]), "x_last": (host(x), xr, 1e-4), "ckpt": (host(ckpt), before, 1e-4)}, disc)
