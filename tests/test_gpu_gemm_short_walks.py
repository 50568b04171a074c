"""Rows added to in 256x128 tiles change their loop at K = 2048: both sides of that line give the bits of the 256x256 tile, at the
edges of the tile, for wrapped walks along K and with a row map."""
import pytest
import torch

from test_gpu_gemm_bits import REFERENCE, RESIDUAL, Product, same_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("K,wrapped", [(64, False), (192, False), (256, True), (1984, False), (2048, False), (2048, True), (2112, False)])
def test_both_loops_give_the_same_bits(K, wrapped, dtype):
    for n, M in enumerate((1, 255, 256, 257, 643)):
        p = Product(dtype, M, 768, K, K // 2 if wrapped else K, RESIDUAL, seed=n)
        assert same_bits(p.run(20), p.run(REFERENCE)), (M, K, wrapped)


@pytest.mark.parametrize("K", [448, 2048])
def test_row_map_and_padding(K):
    rows = torch.randperm(900, device="cuda", dtype=torch.int32)[:265].contiguous()
    p = Product("f16", 265, 256, K, K, RESIDUAL, seed=3, rows=rows, n_valid=253)
    assert same_bits(p.run(20), p.run(REFERENCE))
