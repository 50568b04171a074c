"""Tile choice of the 16-bit MFMA GEMM (radix_debug_gemm_plan, the function the launcher calls): for every size the rows
are split into at most two launches, each with a tile shape its epilogue can run and that divides the output width."""
import ctypes as C
import os

import pytest

from paper_2601_15013_amd import binding

STORE, RESIDUAL, SWIGLU, QKV_ROPE, STORE_F32, SWIGLU_SPLIT, QKV_ROPE_SPLIT = 0, 1, 2, 3, 4, 5, 7


@pytest.fixture(scope="module")
def plan():
    if not os.path.exists(binding.LIB_PATH):
        from paper_2601_15013_amd import build
        build.build()
    lib = binding.load_library()

    def call(*args):
        out = [C.c_int32(-1) for _ in range(7)]
        rc = lib.radix_debug_gemm_plan(*args, *[C.byref(o) for o in out])
        return rc, [o.value for o in out]
    return call


@pytest.mark.parametrize("epilogue", [STORE, RESIDUAL, SWIGLU, QKV_ROPE, STORE_F32, SWIGLU_SPLIT, QKV_ROPE_SPLIT])
def test_every_size_has_a_plan_that_covers_its_rows(plan, epilogue):
    widths = [256, 512, 1024, 4096, 19456] if epilogue in (QKV_ROPE, QKV_ROPE_SPLIT) else [128, 256, 384, 1024, 2560, 19456, 151936]
    seen = set()
    for nout in widths:
        for k in (64, 128, 1024, 3072, 12288, 24576):
            for m in (1, 15, 16, 17, 31, 32, 33, 64, 65, 127, 128, 129, 255, 256, 257, 511, 768, 1072, 2200, 4096, 8191, 8192,
                      8240, 16385, 45120, 266240):
                rc, (v1, bm1, bn1, m1, v2, bm2, bn2) = plan(m, nout, k, epilogue)
                assert rc == 0 and 0 < m1 <= m, (m, nout, k)
                parts = [(v1, bm1, bn1)] + ([(v2, bm2, bn2)] if m1 < m else [])
                if m1 < m:
                    assert m1 % bm1 == 0        # whole tiles in front, so that no row is computed twice
                for v, bm, bn in parts:
                    seen.add(v)
                    assert v > 0 and nout % bn == 0
                    if epilogue in (QKV_ROPE, QKV_ROPE_SPLIT):
                        assert bn % 128 == 0
                    if epilogue in (SWIGLU, SWIGLU_SPLIT):
                        assert bn % 64 == 0
    assert len(seen) >= 5


def test_plan_rejects_bad_sizes(plan):
    assert plan(0, 128, 64, 0)[0] == -2 and plan(8, 128, 0, 0)[0] == -2
