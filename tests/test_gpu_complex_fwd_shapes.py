"""GPU parity of the complex forward pass in each of its launch shapes (16 lanes of 16 steps for many rows, 64 of 8 for some, 64 of 4
for few) at the edges of a lane, a checkpoint interval and a tile, with channel counts that leave lanes without a channel; its
checkpoints by the backward pass that starts from them, and the state-only sweep of a backward pass without any."""
import pytest

import test_gpu_packed_complex as packed
import test_gpu_selective_complex as fwd
import test_gpu_selective_complex_bwd as bwd
from test_gpu_selective_complex import api  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("N,B,D,L,groups", [
    (16, 1, 8201, 17, 1), (1, 1, 8203, 255, 1), (4, 2, 4201, 257, 1), (8, 8, 1025, 256, 1), (16, 2, 4102, 300, 2), (2, 1, 9001, 513, 1),
    (16, 2, 771, 513, 1), (8, 2, 773, 1023, 1), (4, 1, 1602, 520, 3), (1, 2, 777, 1025, 1),
    (16, 1, 5, 255, 1), (8, 3, 7, 257, 1), (4, 1, 2, 9, 1), (2, 1, 3, 260, 1),
    (1, 3, 5003, 255, 1), (2, 2, 6001, 300, 1), (1, 2, 1603, 770, 1)])
def test_launch_shapes(api, oracle, io, N, B, D, L, groups):
    disc = fwd.DISCS[(N + D + L) % 4]
    fwd._run(api, oracle, B, D, N, L, io, disc, gate=True, x0=True, seed=N + L, groups=groups, path="single_pass")


@pytest.mark.parametrize("use_ckpt", [True, False])
@pytest.mark.parametrize("N,B,D,L", [(16, 1, 8201, 270), (2, 2, 771, 1030), (8, 1, 9, 300)])
def test_checkpoints_and_sweep_in_each_shape(api, oracle, N, B, D, L, use_ckpt):
    bwd._run(api, oracle, B, D, N, L, "bf16", "zoh_s6", gate=True, x0=True, seed=N + L, use_ckpt=use_ckpt)


# more chunks than one thread of the carry kernel takes, and more than a workgroup takes at a time
@pytest.mark.parametrize("N,D,L", [(4, 3, 5000), (1, 2, 70000), (16, 40, 9000)])
def test_chunk_carry_chains(api, oracle, N, D, L):
    fwd._run(api, oracle, 1, D, N, L, "f32", "zoh_s6", gate=True, x0=True, seed=L, path="chunk_carry")


# chunks of several tiles: the product of the multipliers and the end state are kept from tile to tile (bilinear: by multiplication),
# the next tile is fetched up to the chunk's end, and the last chunk ends in a ragged tile
@pytest.mark.parametrize("N,disc,io", [(16, "zoh_s6", "f32"), (16, "bilinear", "bf16"), (2, "zoh", "bf16"), (4, "bilinear", "f32")])
def test_chunks_of_several_tiles(api, oracle, N, disc, io):
    B, D, L = 8, 272, 4700
    chunks, tiles = api.lib().lrnnx_selective_scan_fwd_complex_chunks(B, D, N, L, 1, 2), -(-L // 256)
    assert 1 < chunks < tiles, "a plan of several tiles a chunk"
    fwd._run(api, oracle, B, D, N, L, io, disc, gate=True, x0=True, seed=N, path="chunk_carry")


# packed batches in each shape: 24 and 20 short sequences (16 lanes), 3 long ones of many channels (64 x 8), 3 of hardly two tiles (64 x 4)
@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("N,D,lengths", [
    (16, 515, [1, 255, 256, 257] + 20 * [49]), (4, 700, [300, 9] + 18 * [33]), (8, 1001, [511, 513, 1476]), (16, 801, [3, 260, 437])])
def test_packed_shapes(api, oracle, io, N, D, lengths):
    packed._check(api, oracle, D, N, lengths, io, seed=N + D)
