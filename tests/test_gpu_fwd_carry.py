"""GPU parity of the chain over chunk aggregates: chunk counts at the edges of what a thread folds (16 chunks), of what a workgroup
takes at a time (256) and beyond, chains that fill no workgroup, and a start state."""
import pytest

from paper_2602_08810_amd import workloads
from _util import check_outputs, host, sel_inputs_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,D,L", [(1, 1, 511), (4, 3, 4096), (16, 2, 4353), (2, 9, 8192), (8, 1, 65536), (1, 17, 65537), (4, 1, 131400)])
def test_chunk_carry_chain(oracle, N, D, L):
    from paper_2602_08810_amd import api
    p = workloads.make_selective(B=1, D=D, N=N, L=L, io="f32", gate=False, with_x0=True, seed=N + L, bias=("uniform", -7.0, -6.0))
    y, x, ck = api.lrnnx_selective_scan_fwd(**sel_inputs_dev(p, "f32"), return_last_state=True, return_ckpt=True, path="chunk_carry")
    yr, xr, xs = oracle.selective_scan_fwd(**{k: p[k] for k in ("u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "x0")}, return_states=True)
    check = {"y": (host(y), yr, 1e-4), "x_last": (host(x), xr, 1e-4)}
    if L > 256:
        check["ckpt"] = (host(ck)[:, :, 1:], xs[:, :, 255:L - 1:256, :], 1e-4)
    check_outputs(check)
