"""Host-only check (no GPU) of where a forward pass takes twelve channels a workgroup, at calls that were measured in every shape: not where that is
clearly slower, always where it saves much."""
import ctypes
import os

import pytest

from paper_2602_08810_amd import api

LIB = os.path.join(os.path.dirname(api.__file__), "liblrnnx.so")
TWELVE = 4                                                  # 64 lanes of 8 steps, twelve wavefronts

# (maps, channels of a map, N, L, float32[, states alone]): the best other shape, twelve channels (us, or the former as 1)
SLOWER = [((1, 2600, 16, 768, True), 20.1, 23.1), ((1, 2049, 32, 768, True), 29.1, 37.3), ((1, 2600, 8, 1280, True), 20.1, 22.7),
          ((1, 2600, 32, 513, True), 34.3, 36.3), ((1, 2049, 8, 5000, True), 53.3, 57.8), ((3, 683, 32, 1280, True), 1.0, 1.15),
          ((9, 228, 8, 1280, False), 1.0, 1.12), ((3, 683, 8, 1792, True), 1.0, 1.11), ((1, 2051, 8, 3000, False), 1.0, 1.05), ((1, 2200, 8, 768, True, True), 1.0, 1.16),
          ((3, 771, 16, 700, False, True), 1.0, 1.08), ((1, 2049, 16, 3000, True, True), 1.0, 1.09)]
FASTER = [((1, 2064, 16, 1536, False), 30.9, 26.8), ((1, 2600, 32, 12000, False), 1.0, 0.81), ((3, 683, 16, 3000, True), 1.0, 0.86),
          ((1, 3072, 8, 400, True), 1.0, 0.95), ((2, 1025, 32, 1024, False), 1.0, 0.84), ((1, 2053, 16, 1281, True), 1.0, 0.88),
          ((5, 410, 32, 1792, False), 1.0, 0.93), ((33, 63, 16, 5000, True), 1.0, 0.84),
          ((1, 2800, 32, 1280, True, True), 1.0, 0.91), ((3, 771, 16, 1100, True, True), 1.0, 0.98), ((1, 2200, 32, 2048, False, True), 1.0, 0.83)]


@pytest.mark.parametrize("call,other,twelve", SLOWER + FASTER)
def test_twelve_channels(call, other, twelve):
    if not os.path.exists(LIB):
        pytest.skip("liblrnnx.so not built")
    shape = ctypes.CDLL(LIB)._ZN5lrnnx16fwd_shape_numberEllllbb           # lrnnx::fwd_shape_number
    got = shape(*(ctypes.c_int64(n) for n in call[:4]), ctypes.c_bool(call[4]), ctypes.c_bool(not call[5:]))
    assert (got == TWELVE) == (twelve < other), got


def test_only_where_it_fits():
    if not os.path.exists(LIB):
        pytest.skip("liblrnnx.so not built")
    shape = ctypes.CDLL(LIB)._ZN5lrnnx16fwd_shape_numberEllllbb
    for maps, dpg, N in ((1, 2048, 16), (1, 3073, 16), (257, 1, 16), (1, 2600, 4), (300, 8, 16)):
        for L in (1, 400, 1536, 9000):
            for f32 in (False, True):
                assert shape(*(ctypes.c_int64(n) for n in (maps, dpg, N, L)), ctypes.c_bool(f32), ctypes.c_bool(True)) != TWELVE
