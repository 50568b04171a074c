"""Every tile of the 16-bit products gives the same bits: a row's result must not depend on which tile its batch size picks,
so all (tile, epilogue) pairs that a plan can choose are compared with the eight-wavefront 256x256 tile on the same
operands, at the edges of the tile and for short, odd and wrapped walks along K - and that tile with float64."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2601_15013_amd import binding

pytestmark = pytest.mark.gpu

STORE, RESIDUAL, SWIGLU, QKV_ROPE, STORE_F32, SWIGLU_SPLIT, QKV_ROPE_SPLIT = 0, 1, 2, 3, 4, 5, 7
EPILOGUES = [STORE, RESIDUAL, SWIGLU, QKV_ROPE, STORE_F32, SWIGLU_SPLIT, QKV_ROPE_SPLIT]
ROPE = (QKV_ROPE, QKV_ROPE_SPLIT)
TILES = {4: (256, 256), 11: (32, 16), 12: (32, 32), 13: (32, 128), 14: (32, 64), 15: (64, 32), 16: (64, 64),
         17: (64, 128), 18: (128, 128), 19: (128, 256), 20: (256, 128)}
DTYPES = {"f16": (torch.float16, 2), "bf16": (torch.bfloat16, 1)}
REFERENCE = 4


def usable(tile, epilogue):
    bn = TILES[tile][1]
    if epilogue in ROPE:
        return bn % 128 == 0
    return bn % 64 == 0 if epilogue in (SWIGLU, SWIGLU_SPLIT) else True


class Product:
    """Operands of one product, and its result in any tile."""

    def __init__(self, dtype, M, nout, K, w_k, epilogue, seed=0, a=None, w=None, rows=None, n_valid=0):
        self.t, self.code = DTYPES[dtype]
        self.M, self.nout, self.K, self.w_k, self.epi = M, nout, K, w_k, epilogue
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        self.rows, self.n_valid = rows, n_valid
        self.n_src = M if rows is None else int(rows.max()) + 1
        rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)  # noqa: E731
        self.A = rnd(self.n_src, K).to(self.t) if a is None else a
        self.W = (rnd(nout, w_k) * 0.05).to(self.t) if w is None else w
        self.gq, self.gk = 1 + 0.1 * rnd(128), 1 + 0.1 * rnd(128)
        angle = torch.arange(64, device="cuda")[:, None] * torch.logspace(0, -3, 64, device="cuda")[None]
        self.cos, self.sin = angle.cos().contiguous(), angle.sin().contiguous()
        self.pos = ((torch.arange(M, device="cuda", dtype=torch.int32) * 7) % 64).to(torch.int32)
        self.resid = rnd(M, nout)
        self.status = torch.zeros(1, dtype=torch.int32, device="cuda")
        self.kv = nout // 128 // 4 if epilogue in ROPE else 0
        self.q = nout // 128 - 2 * self.kv if epilogue in ROPE else 0

    def run(self, tile):
        if self.epi == RESIDUAL:
            out = self.resid.clone()
        else:
            width = {STORE: self.nout, QKV_ROPE: self.nout, STORE_F32: self.nout, SWIGLU: self.nout // 2, SWIGLU_SPLIT: self.nout,
                     QKV_ROPE_SPLIT: 2 * self.nout}[self.epi]
            out = torch.full((self.M + 1, width), 77.0, dtype=torch.float32 if self.epi == STORE_F32 else self.t, device="cuda")
        p = lambda t: None if t is None else t.data_ptr()  # noqa: E731
        rc = binding.load_library().radix_debug_gemm_run(
            p(self.A), p(self.W), self.M, self.nout, self.K, self.w_k, self.epi, p(out), self.code, tile, p(self.gq), p(self.gk),
            p(self.cos), p(self.sin), p(self.pos), self.q, self.kv, 1, p(self.rows), self.n_valid, self.n_src, p(self.status),
            torch.cuda.current_stream().cuda_stream)
        assert rc == 0, rc
        assert int(self.status.item()) == 0
        if self.epi != RESIDUAL:
            assert bool((out[self.M] == 77.0).all()), "the row past the end was written"
            out = out[:self.M]
        return out


def same_bits(a, b):
    """Bit for bit; a NaN may be any NaN."""
    ints = {4: torch.int32, 2: torch.int16}[a.element_size()]
    return bool(((a.view(ints) == b.view(ints)) | (a.isnan() & b.isnan())).all())


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("tile,epilogue", [(t, e) for t in sorted(TILES) if t != REFERENCE for e in EPILOGUES if usable(t, e)])
def test_every_tile_gives_the_same_bits(tile, epilogue, dtype):
    bm = TILES[tile][0]
    # K in k-tiles of 64: one, two, an odd number below, at and above the depth of every ring of stages (3 to 8), and many
    for n, (K, wrapped) in enumerate([(64, False), (128, True), (192, False), (448, False), (512, False), (576, False), (640, True),
                                      (1088, False), (2176, True)]):
        M = [1, bm - 1, bm, bm + 1, 2 * bm + 3, 3 * bm - 1, 17, bm // 2 + 5, 300][n]
        p = Product(dtype, M, 768, K, K // 2 if wrapped else K, epilogue, seed=n)
        assert same_bits(p.run(tile), p.run(REFERENCE)), (M, K, wrapped)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("epilogue", EPILOGUES)
def test_the_reference_tile_against_float64(epilogue, dtype):
    M, K, nout = 259, 576, 768
    p = Product(dtype, M, nout, K, K, epilogue, seed=3)
    got = p.run(REFERENCE).cpu().double()
    c = p.A.cpu().double() @ p.W.cpu().double().T
    parts = 1
    if epilogue == RESIDUAL:
        want = p.resid.cpu().double() + c
    elif epilogue in (SWIGLU, SWIGLU_SPLIT):
        c = c.view(M, nout // 64, 2, 32)
        want = (torch.nn.functional.silu(c[:, :, 0]) * c[:, :, 1]).reshape(M, nout // 2)
        parts = 1 + (epilogue == SWIGLU_SPLIT)
    elif epilogue in ROPE:
        parts = 1 + (epilogue == QKV_ROPE_SPLIT)
        h = c.view(M, nout // 128, 128)
        want = h.clone()
        gain = torch.cat([p.gq.cpu().double().expand(p.q, 128), p.gk.cpu().double().expand(p.kv, 128)])
        n = h[:, :p.q + p.kv]
        n = n * torch.rsqrt((n * n).mean(-1, keepdim=True) + 1e-6) * gain
        cs, sn = (t.cpu().double()[p.pos.cpu().long()][:, None] for t in (p.cos, p.sin))
        want[:, :p.q + p.kv] = torch.cat([n[..., :64] * cs - n[..., 64:] * sn, n[..., 64:] * cs + n[..., :64] * sn], -1)
        want = want.reshape(M, nout)
    else:
        want = c
    if parts == 2:
        got = got[:, :want.shape[1]] + got[:, want.shape[1]:]
    # fp32 sums of K products (each partial sum below the sum of magnitudes), which the head's norm and the gate may scale by a
    # few; a 16-bit result adds its own half unit, a (hi, lo) pair the square of that (fp16: half a unit of its sub-normals)
    mag = (p.A.cpu().double().abs() @ p.W.cpu().double().abs().T).max()
    ulp = {"f16": 2.0 ** -11, "bf16": 2.0 ** -8}[dtype]
    rel = 0.0 if epilogue in (RESIDUAL, STORE_F32) else (ulp if parts == 1 else ulp * ulp + 2.0 ** -24)
    scale = float(want.abs().max()) if epilogue in (SWIGLU, SWIGLU_SPLIT) + ROPE else float(mag)
    err = (got - want).abs()
    assert bool((err <= 8 * K * 2.0 ** -24 * scale + rel * (want.abs() + 1.0)).all()), float(err.max())


@pytest.mark.parametrize("kind", ["wide", "subnormal", "inf", "nan", "huge", "overflow"])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_special_operands_give_the_same_bits_in_every_tile(dtype, kind):
    # one 16x16x32 matrix instruction must round like two 32x32x16 ones on every operand, not only on well-behaved ones
    t, _ = DTYPES[dtype]
    M, nout, K = 70, 256, 320
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    a, w = torch.randn(M, K, device="cuda", generator=g), torch.randn(nout, K, device="cuda", generator=g)
    tiny, big = (2.0 ** -24, 6e4) if dtype == "f16" else (2.0 ** -133, 3e38)
    e = 12 if dtype == "f16" else 60
    if kind == "wide":          # exponents all over the range: most products vanish beside others of the same sum
        a *= torch.exp2(torch.randint(-e, e // 4, (M, K), device="cuda", generator=g).float())
        w *= torch.exp2(torch.randint(-e, e // 4, (nout, K), device="cuda", generator=g).float())
    elif kind == "subnormal":
        a = torch.randint(-40, 41, (M, K), device="cuda", generator=g).double().mul(tiny).float()
        w *= 0.05 if dtype == "f16" else 2.0 ** -14
    elif kind == "inf":
        a[torch.rand(M, K, device="cuda", generator=g) < 0.01] = float("inf")
        a[torch.rand(M, K, device="cuda", generator=g) < 0.01] = float("-inf")
        w[torch.rand(nout, K, device="cuda", generator=g) < 0.01] = 0.0
    elif kind == "nan":
        a[torch.rand(M, K, device="cuda", generator=g) < 0.002] = float("nan")
    elif kind == "overflow":    # finite products whose running sums leave fp32 and may come back (bf16)
        a, w = a.sign(), w.sign() * (1.5e38 if dtype == "bf16" else 6e4)
    else:                       # products that overflow fp32 (bf16) or the 16-bit result (fp16)
        a, w = a.sign() * big, w.sign() * (big if dtype == "bf16" else 60.0)
        a[torch.rand(M, K, device="cuda", generator=g) < 0.7] = 1.0
    a, w = a.to(t), w.to(t)
    for epilogue in (STORE, RESIDUAL, SWIGLU, STORE_F32, SWIGLU_SPLIT):
        p = Product(dtype, M, nout, K, K, epilogue, a=a, w=w)
        ref = p.run(REFERENCE)
        for tile in sorted(TILES):
            if usable(tile, epilogue):
                assert same_bits(p.run(tile), ref), (tile, epilogue)


def split_of(M, nout, K, epilogue):
    out = [C.c_int32(-1) for _ in range(7)]
    assert binding.load_library().radix_debug_gemm_plan(M, nout, K, epilogue, *[C.byref(o) for o in out]) == 0
    return out[3].value


@pytest.mark.parametrize("n_valid", ["all", "past the cut", "at the cut", "before the cut", "none"])
def test_a_split_product_reads_its_rows_through_the_map(n_valid):
    # rows through an index map, the last ones padding, in a product whose plan cuts the rows in two launches
    M, nout, K = 8240, 1024, 2048
    cut = split_of(M, nout, K, RESIDUAL)
    assert 0 < cut < M
    valid = {"all": M, "past the cut": (cut + M) // 2, "at the cut": cut, "before the cut": cut - 301, "none": 0}[n_valid]
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    rows = torch.randint(0, 9000, (M,), device="cuda", generator=g, dtype=torch.int32)
    rows[0] = 8999
    rows[valid:] = 8999                 # what the map holds for padding rows is not read
    p = Product("f16", M, nout, K, K, RESIDUAL, rows=rows, n_valid=valid)
    got = p.run(0)
    assert same_bits(got, p.run(REFERENCE))
    picked = torch.where(torch.arange(M, device="cuda") < valid, rows, torch.zeros_like(rows)).long()
    q = Product("f16", M, nout, K, K, RESIDUAL, a=p.A[picked].contiguous(), w=p.W)
    q.resid = p.resid
    assert same_bits(got, q.run(REFERENCE))


@pytest.mark.parametrize("epilogue", EPILOGUES)
def test_a_split_product_equals_the_unsplit_one(epilogue):
    nout, K = (4096, 1024) if epilogue in ROPE else (1024, 3072)
    for M in (8240, 8672, 16436):
        if split_of(M, nout, K, epilogue) == M:
            continue
        p = Product("f16", M, nout, K, K, epilogue, seed=M)
        assert same_bits(p.run(0), p.run(REFERENCE)), M
        return
    pytest.fail("no split at these sizes")


def test_the_hook_refuses_what_the_tiles_cannot_run():
    p = Product("f16", 8, 256, 64, 64, STORE)
    for tile, epilogue in ((1, STORE), (1, RESIDUAL), (2, STORE), (3, SWIGLU), (99, STORE), (16, QKV_ROPE), (15, SWIGLU)):
        p.epi = epilogue
        out = torch.zeros(8, 512, dtype=torch.float32, device="cuda")
        q = (lambda t: t.data_ptr())
        rc = binding.load_library().radix_debug_gemm_run(q(p.A), q(p.W), 8, 256, 64, 64, epilogue, q(out), 2, tile, q(p.gq), q(p.gk),
                                                         q(p.cos), q(p.sin), q(p.pos), 0, 1, 1, None, 0, 8, None, 0)
        assert rc == -3
        assert np.all(out.cpu().numpy() == 0)
