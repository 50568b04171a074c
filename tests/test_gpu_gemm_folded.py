"""The tiles of products with a folded RMSNorm.  A consumed norm whose row scales are powers of two is the plain product of scaled
rows, bit for bit, in every tile; with other scales all tiles give the same bits, near float64.  A prepared norm leaves the residual
rows of the plain product, their product with the gain in the operand type, and sums of squares that do not depend on the tile."""
import ctypes as C

import pytest
import torch

from paper_2601_15013_amd import binding
from test_gpu_gemm_bits import QKV_ROPE, REFERENCE, RESIDUAL, STORE, SWIGLU, Product, same_bits

pytestmark = pytest.mark.gpu

PREPARE = 6
ROWS = {1: 256, 2: 128, 3: 128, 4: 256}
CONSUMERS = [(4, STORE), (4, SWIGLU), (4, QKV_ROPE), (3, STORE), (3, SWIGLU), (3, QKV_ROPE), (2, STORE), (2, SWIGLU)]
# K in k-tiles of 64: below, at and above the depth of every ring of stages
LENGTHS = [64, 128, 192, 256, 320, 576, 1088]


def rows_of(bm):
    return [1, bm - 1, bm, bm + 1, 2 * bm + 3, bm // 2 + 5, 3 * bm - 17]


def run(p, tile, epilogue, ss=None, inv_d=1.0, eps=0.0, out=None, a16=None, gain=None, ss_out=None):
    ptr = lambda t: None if t is None else t.data_ptr()  # noqa: E731
    if out is None:
        out = torch.full((p.M + 1, p.nout // 2 if epilogue == SWIGLU else p.nout), 77.0, dtype=p.t, device="cuda")
    rc = binding.load_library().radix_debug_gemm_run_folded(
        ptr(p.A), ptr(p.W), p.M, p.nout, p.K, epilogue, ptr(out), p.code, tile, ptr(p.gq), ptr(p.gk), ptr(p.cos), ptr(p.sin), ptr(p.pos),
        p.q, p.kv, ptr(ss), 0 if ss is None else ss.shape[1], inv_d, eps, ptr(a16), ptr(gain), ptr(ss_out),
        torch.cuda.current_stream().cuda_stream)
    assert rc == 0, rc
    assert epilogue == PREPARE or bool((out[p.M] == 77.0).all()), "the row past the end was written"
    return out[:p.M]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("tile,epilogue", CONSUMERS)
def test_scales_that_are_powers_of_two(tile, epilogue, dtype):
    for n, K in enumerate(LENGTHS):
        M, slots = rows_of(ROWS[tile])[n], (2, 6, 8, 16, 18, 34, 40)[n]
        p = Product(dtype, M, 768, K, K, epilogue, seed=n)
        e = torch.arange(M, device="cuda") % 5 - 2                      # scales 1/4 .. 4
        ss = torch.zeros(M, slots, device="cuda")
        ss[torch.arange(M), torch.arange(M) % slots] = torch.exp2(-2.0 * e.float())
        p.A[p.A.abs() < 2.0 ** -8] = 0                                  # a quarter of the others is exact in fp16
        q = Product(dtype, M, 768, K, K, epilogue, seed=n)
        q.A = (p.A.float() * torch.exp2(e.float())[:, None]).to(p.t)
        assert same_bits(run(p, tile, epilogue, ss), q.run(REFERENCE)), (M, K, slots)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("epilogue", [STORE, SWIGLU, QKV_ROPE])
def test_any_scales_give_the_same_bits_in_every_tile(epilogue, dtype):
    for n, K in enumerate(LENGTHS):
        M, slots = (1, 130, 255, 300, 515, 700, 31)[n], (2, 6, 8, 16, 18, 34, 40)[n]
        p = Product(dtype, M, 768, K, K, epilogue, seed=n)
        ss = torch.rand(M, slots, device="cuda") * 300
        inv_d = 1.0 / (128 * slots)
        got = run(p, 4, epilogue, ss, inv_d, 1e-6)
        for tile, e in CONSUMERS:
            if e == epilogue and tile != 4:
                assert same_bits(run(p, tile, epilogue, ss, inv_d, 1e-6), got), (tile, M, K)
        assert same_bits(run(p, 0, epilogue, ss, inv_d, 1e-6), got), (M, K)
        if epilogue == STORE:
            scale = (ss.double().sum(1, keepdim=True) * inv_d + 1e-6).rsqrt()
            want = (p.A.double() @ p.W.double().T.contiguous()) * scale
            mag = (p.A.double().abs() @ p.W.double().abs().T.contiguous()) * scale
            # fp32 sums of K products, of the slots and one square root, then half a unit of the operand type (or its sub-normals)
            bound = (K + slots + 8) * 2.0 ** -24 * mag + {"f16": 2.0 ** -11, "bf16": 2.0 ** -8}[dtype] * want.abs() + 2.0 ** -24
            assert bool(((got.double() - want).abs() <= bound).all()), (M, K)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("tile", [1, 3, 0])
def test_a_prepared_norm(tile, dtype):
    for n, K in enumerate(LENGTHS):
        M = rows_of(ROWS.get(tile, 256))[n]
        p = Product(dtype, M, 768, K, K, RESIDUAL, seed=n)
        gain = 1 + 0.1 * torch.randn(768, device="cuda")
        a16 = torch.full((M + 1, 768), 77.0, dtype=p.t, device="cuda")
        ss = torch.full((M + 1, 6), 77.0, device="cuda")
        out = run(p, tile, PREPARE, out=torch.cat([p.resid, torch.full((1, 768), 77.0, device="cuda")]), a16=a16, gain=gain, ss_out=ss)
        assert bool((a16[M] == 77.0).all()) and bool((ss[M] == 77.0).all()), "a row past the end was written"
        assert same_bits(out, p.run(REFERENCE)), (M, K)
        assert same_bits(a16[:M], (out * gain).to(p.t)), (M, K)
        want = (out.double() ** 2).view(M, 6, 128).sum(-1)
        assert bool(((ss[:M].double() - want).abs() <= 128 * 2.0 ** -24 * want).all()), (M, K)
        other = torch.empty_like(ss)
        run(p, 4 - tile if tile else 1, PREPARE, out=p.resid.clone(), a16=a16, gain=gain, ss_out=other)
        assert torch.equal(other[:M], ss[:M]), (M, K)


def test_what_the_folded_tiles_refuse():
    lib = binding.load_library()
    p = Product("f16", 8, 256, 64, 64, STORE)
    buf, ss = torch.zeros(8, 512, device="cuda"), torch.ones(8, 4, device="cuda")
    ptr = lambda t: t.data_ptr()  # noqa: E731

    def call(tile, epilogue, slots=4, given=ss):
        return lib.radix_debug_gemm_run_folded(ptr(p.A), ptr(p.W), 8, 256, 64, epilogue, ptr(buf), 2, tile, ptr(p.gq), ptr(p.gk), ptr(p.cos),
                                               ptr(p.sin), ptr(p.pos), 0, 1, None if given is None else ptr(given), slots, 1.0, 0.0,
                                               ptr(buf), ptr(p.resid), ptr(buf), C.c_void_p(0))

    for tile, epilogue in ((1, STORE), (1, QKV_ROPE), (2, QKV_ROPE), (2, PREPARE), (4, PREPARE), (5, STORE), (20, STORE), (4, 4), (4, 1), (4, 5)):
        assert call(tile, epilogue) == -3, (tile, epilogue)
    assert call(4, STORE, slots=3) == -3 and call(4, STORE, slots=0) == -3 and call(4, STORE, given=None) == -1
    torch.cuda.synchronize()
    assert not bool(buf.any())
