"""GPU parity of the sums of dBm and dCm of packed batches around the sizes where four threads share an element."""
import pytest

from test_gpu_packed import _check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2602_08810_amd import api as _api
    _api.lib()
    return _api


# 16-state slots have 8 workgroups and 32-state ones 16: below three halves of the chip, between that and three a CU, beyond it; short last
# tiles and empty sequences
@pytest.mark.parametrize("N,lengths", [
    (16, [2048] * 4), (16, [1900, 0, 2049, 2048, 1, 2047, 2305, 2500]), (16, [2048] * 12), (32, [1023, 1025, 0, 2048, 1000]), (8, [2048] * 14),
    (8, [2000, 0] * 12)])
def test_packed_sums(api, oracle, N, lengths):
    _check(api, oracle, 640, N, lengths, "f32", seed=N * 31 + len(lengths))
