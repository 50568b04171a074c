"""The tiles whose rows are no power of two (160, 192 and 224) give the bits of the 256x256 tile: at the edges of the tile, for
short, odd and wrapped walks along K, with a row map whose last rows are padding, and where the rows of A do not share out
evenly over the wavefronts' loads."""
import pytest
import torch

from test_gpu_gemm_bits import EPILOGUES, QKV_ROPE, QKV_ROPE_SPLIT, REFERENCE, RESIDUAL, Product, same_bits

pytestmark = pytest.mark.gpu

ROWS = {22: 160, 23: 192, 24: 224}


def usable(tile, epilogue):
    return epilogue not in (QKV_ROPE, QKV_ROPE_SPLIT) or tile == 23


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("tile,epilogue", [(t, e) for t in ROWS for e in EPILOGUES if usable(t, e)])
def test_tiles_of_other_heights_give_the_same_bits(tile, epilogue, dtype):
    bm = ROWS[tile]
    for n, (K, wrapped) in enumerate([(64, False), (128, True), (192, False), (320, False), (512, False), (640, True), (2176, True)]):
        M = [1, bm - 1, bm, bm + 1, 2 * bm + 3, bm // 2 + 5, 3 * bm - 17][n]
        p = Product(dtype, M, 768, K, K // 2 if wrapped else K, epilogue, seed=n)
        assert same_bits(p.run(tile), p.run(REFERENCE)), (M, K, wrapped)


@pytest.mark.parametrize("tile", sorted(ROWS))
def test_row_map_and_padding(tile):
    M, valid = ROWS[tile] + 9, ROWS[tile] - 3
    rows = torch.randperm(700, device="cuda", dtype=torch.int32)[:M].contiguous()
    p = Product("f16", M, 256, 448, 448, RESIDUAL, seed=3, rows=rows, n_valid=valid)
    assert same_bits(p.run(tile), p.run(REFERENCE))


def test_split_tiles_without_whole_heads_refuse_the_head_epilogue():
    for tile in (22, 24):
        with pytest.raises(AssertionError):
            Product("f16", 64, 768, 64, 64, QKV_ROPE).run(tile)
