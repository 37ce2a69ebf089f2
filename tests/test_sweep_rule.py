"""Host-only check (no GPU) of the rule that cuts the forward sweep of a backward call without checkpoints into chunks of the time axis, at calls that
were measured both ways: never where that is clearly slower than one chain a row, always where it saves much."""
import ctypes
import os

import pytest

from paper_2602_08810_amd import api

LIB = os.path.join(os.path.dirname(api.__file__), "liblrnnx.so")

# (B, groups, channels of a group, N, L, float32): one chain, in chunks (us)
SLOWER = [((1, 1, 1024, 32, 4096, False), 50.6, 61.6), ((1, 1, 1536, 32, 16384, True), 238.7, 270.7), ((1, 1, 1024, 16, 8192, False), 52.5, 59.5),
          ((1, 1, 512, 16, 2048, False), 15.8, 17.9), ((1, 1, 384, 16, 2048, False), 15.7, 17.6), ((1, 1, 16, 16, 2048, False), 15.4, 16.7),
          ((1, 1, 1024, 16, 4096, True), 34.3, 38.1), ((1, 1, 1024, 32, 4096, True), 62.1, 67.0), ((3, 1, 1, 16, 1945, False), 13.2, 16.8),
          ((4, 2, 2, 4, 2237, False), 9.5, 12.0), ((6, 2, 186, 16, 17456, False), 182.8, 221.5), ((4, 1, 4, 16, 1859, False), 14.2, 16.1)]
FASTER = [((1, 1, 16, 16, 65536, False), 390.2, 18.6), ((1, 1, 16, 16, 65536, True), 489.5, 19.5), ((1, 1, 256, 16, 4096, False), 27.7, 17.8),
          ((1, 1, 768, 16, 16384, False), 101.0, 81.3), ((1, 1, 64, 4, 65536, False), 170.1, 19.9), ((1, 1, 1024, 32, 65536, True), 1012.2, 711.0),
          ((1, 1, 512, 8, 8192, True), 40.7, 27.5), ((1, 1, 128, 1, 16384, False), 26.0, 12.0)]


@pytest.mark.parametrize("call,chain,chunks", SLOWER + FASTER)
def test_rule(call, chain, chunks):
    if not os.path.exists(LIB):
        pytest.skip("liblrnnx.so not built")
    pays = ctypes.CDLL(LIB)._ZN5lrnnx16sweep_chunks_payElllllb          # lrnnx::sweep_chunks_pay
    pays.restype = ctypes.c_bool
    assert pays(*(ctypes.c_int64(n) for n in call[:5]), ctypes.c_bool(call[5])) == (chunks < chain)


def test_many_rows_stay_one_chain():
    if not os.path.exists(LIB):
        pytest.skip("liblrnnx.so not built")
    pays = ctypes.CDLL(LIB)._ZN5lrnnx16sweep_chunks_payElllllb
    pays.restype = ctypes.c_bool
    for B, dpg in ((1, 2049), (3, 700), (257, 1), (16, 2560)):
        for L in (256, 257, 5000, 1 << 20, 1 << 31):
            assert not pays(*(ctypes.c_int64(n) for n in (B, 1, dpg, 16, L)), ctypes.c_bool(False))
