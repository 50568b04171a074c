"""Tile choice of the 16-bit MFMA GEMM (radix_debug_gemm_plan, the function the launcher calls): for every size the rows
are split into at most two launches, each with a tile shape its epilogue can run and that divides the output width."""
import ctypes as C
import os

import pytest

from paper_2601_15013_amd import binding

STORE, RESIDUAL, SWIGLU, QKV_ROPE, STORE_F32, SWIGLU_SPLIT, RESIDUAL_NORM, QKV_ROPE_SPLIT = range(8)


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


# rows and widths of the projections (output projection, down, gate/up, q|k|v) of the 0.6B, 4B and 8B shapes
PROJECTIONS = [(1024, 2048, RESIDUAL), (1024, 3072, RESIDUAL), (6144, 1024, SWIGLU), (4096, 1024, QKV_ROPE),
               (2560, 4096, RESIDUAL), (2560, 9728, RESIDUAL), (19456, 2560, SWIGLU), (6144, 2560, QKV_ROPE),
               (4096, 4096, RESIDUAL), (4096, 12288, RESIDUAL), (24576, 4096, SWIGLU), (6144, 4096, QKV_ROPE)]
# rows of a tile
VARIANTS = {4: 256, 11: 32, 12: 32, 13: 32, 14: 32, 15: 64, 16: 64, 17: 64, 18: 128, 19: 128, 20: 256, 22: 160, 23: 192, 24: 224}


def test_plan_is_the_fastest_that_the_cost_model_knows(plan):
    lib = binding.load_library()

    def us(m, nout, k, epi, v1, m1, v2):
        t = C.c_double(-1.0)
        rc = lib.radix_debug_gemm_plan_us(m, nout, k, epi, v1, m1, v2, C.byref(t))
        return t.value if rc == 0 else float("inf")

    for nout, k, epi in PROJECTIONS:
        for m in list(range(257, 20000, 223)) + [7916, 9216, 8672, 939, 658, 33792, 50645]:
            rc, (v1, bm1, _, m1, v2, bm2, _) = plan(m, nout, k, epi)
            assert rc == 0
            assert bm1 == VARIANTS[v1] and (m1 == m or bm2 == VARIANTS[v2]), (m, nout, k)      # the tile named is the tile meant
            t = us(m, nout, k, epi, v1, m1, v2)
            whole = min(us(m, nout, k, epi, v, m, 0) for v in VARIANTS)
            assert t == whole if m1 == m else t < 0.97 * whole, (m, nout, k)
            # no other tile in either part of the chosen split is faster (in the first part: of those that divide its rows)
            for v, bm in VARIANTS.items():
                assert (m1 < m and m1 % bm) or us(m, nout, k, epi, v, m1, v2) >= t, (m, nout, k, v1, v)
                if m1 < m:
                    assert us(m, nout, k, epi, v1, m1, v) >= t, (m, nout, k, v2, v)


def test_plan_counts_the_cus_of_the_device(plan):
    # a partition with the CUs of one XCD: its rounds are full with an eighth of the rows, and tiles grow accordingly
    lib = binding.load_library()

    def on(cus, *args):
        out = [C.c_int32(-1) for _ in range(7)]
        assert lib.radix_debug_gemm_plan_cus(cus, *args, *[C.byref(o) for o in out]) == 0
        return [o.value for o in out]

    for nout, k, epi in PROJECTIONS:
        for m in (939, 1072, 2200, 8672):
            assert on(256, m, nout, k, epi) == plan(m, nout, k, epi)[1]         # no device here: the whole chip
    one, chip = on(32, 939, 1024, 3072, RESIDUAL), on(256, 939, 1024, 3072, RESIDUAL)
    assert one[1] * one[2] > chip[1] * chip[2]
    # 1072 rows of N 4096: 4 row tiles of 256 are two whole rounds of 32 CUs, and 48 rows are left
    v1, bm1, bn1, m1, v2, bm2, bn2 = on(32, 1072, 4096, 4096, RESIDUAL)
    assert m1 == 1024 and bm2 <= 64
    assert lib.radix_debug_gemm_plan_cus(0, 8, 128, 64, 0, *[C.byref(C.c_int32()) for _ in range(7)]) == -2


# us per launch of every usable tile on one MI355X (fp16 operands): products whose rows of A are short, so that most of a launch
# is its epilogue and start-up
SHORT_K = {
    (16500, 384, 128, STORE): {11: 27.19, 12: 19.96, 13: 10.14, 14: 13.48, 15: 14.41, 16: 10.33, 17: 8.43, 18: 9.03, 20: 6.78},
    (50000, 128, 64, RESIDUAL): {11: 27.15, 12: 19.81, 13: 10.94, 14: 14.93, 15: 15.68, 16: 12.78, 17: 9.42, 18: 10.85,
                                 20: 9.45},
    (24000, 128, 128, RESIDUAL): {11: 18.93, 12: 12.07, 13: 7.49, 14: 8.11, 15: 9.92, 16: 7.34, 17: 6.67, 18: 6.95, 20: 8.39},
    (50000, 128, 128, SWIGLU): {13: 9.41, 14: 12.56, 16: 9.31, 17: 7.95, 18: 8.26, 20: 5.89},
    (9216, 256, 256, RESIDUAL): {4: 21.70, 11: 18.58, 12: 13.48, 13: 7.91, 14: 8.67, 15: 11.66, 16: 7.65, 17: 7.30, 18: 7.48,
                                 19: 9.40, 20: 9.47, 22: 14.38, 23: 16.54, 24: 18.54},
    (6500, 384, 384, RESIDUAL): {11: 23.45, 12: 15.01, 13: 9.60, 14: 10.92, 15: 13.15, 16: 10.23, 17: 8.60, 18: 8.43,
                                 20: 11.06},
    (5000, 512, 512, RESIDUAL): {4: 25.53, 11: 28.01, 12: 18.49, 13: 10.58, 14: 13.01, 15: 17.14, 16: 12.58, 17: 9.50,
                                 18: 9.36, 19: 12.02, 20: 12.40, 22: 17.30, 23: 19.85, 24: 22.28},
    (33000, 640, 256, SWIGLU): {13: 31.32, 14: 45.02, 16: 28.93, 17: 23.87, 18: 27.14, 20: 19.26},
    (50000, 4096, 256, STORE_F32): {4: 258.90, 11: 868.03, 12: 681.55, 13: 308.73, 14: 436.30, 15: 427.77, 16: 276.63,
                                    17: 240.12, 18: 299.58, 19: 269.80, 20: 279.84, 22: 307.86, 23: 288.55, 24: 263.45},
    (24000, 4096, 512, STORE_F32): {4: 152.58, 11: 580.75, 12: 462.51, 13: 228.76, 14: 307.87, 15: 295.20, 16: 206.86,
                                    17: 166.45, 18: 181.10, 19: 185.87, 20: 182.67, 22: 179.53, 23: 164.64, 24: 152.84},
    (24000, 384, 384, RESIDUAL): {11: 52.32, 12: 42.93, 13: 23.98, 14: 29.53, 15: 29.17, 16: 23.11, 17: 20.87, 18: 27.49,
                                  20: 26.41},
    (6000, 512, 512, RESIDUAL): {4: 25.95, 11: 33.51, 12: 21.49, 13: 11.26, 14: 15.16, 15: 19.84, 16: 14.39, 17: 10.72,
                                 18: 10.84, 19: 12.44, 20: 13.37, 22: 17.73, 23: 20.14, 24: 22.78},
    (8700, 3072, 512, SWIGLU): {4: 34.51, 13: 59.08, 14: 83.27, 16: 54.25, 17: 41.13, 18: 46.77, 19: 43.91, 20: 38.86,
                                22: 34.86, 23: 38.55, 24: 32.22},
    (3300, 3840, 640, SWIGLU): {4: 20.87, 13: 36.99, 14: 49.36, 16: 33.13, 17: 28.04, 18: 35.38, 19: 26.73, 20: 22.40,
                                22: 25.80, 23: 29.73, 24: 20.02},
}


@pytest.mark.parametrize("product", sorted(SHORT_K))
def test_short_rows_get_a_tile_near_the_best_measured_one(plan, product):
    rc, (v1, _, _, m1, _, _, _) = plan(*product)
    assert rc == 0 and m1 == product[0]
    assert SHORT_K[product][v1] <= 1.1 * min(SHORT_K[product].values())


# us of products of 8 to 20 rounds of workgroups on one MI355X (fp16 operands), by (tile, its rows, tile of the rows left): every large
# tile alone, and with its last, partly filled round given to smaller ones
MANY_ROUNDS = {
    (16436, 6144, 2560, QKV_ROPE): {(4, 16384, 13): 425.5, (4, 16436, 0): 444.2, (18, 16384, 13): 560.7, (18, 16436, 0): 563.1,
        (19, 16384, 13): 523.0, (19, 16436, 0): 525.5, (20, 16384, 13): 529.5, (20, 16436, 0): 526.6, (23, 14208, 4): 436.6,
        (23, 16436, 0): 453.4},
    (24763, 6144, 1024, SWIGLU): {(4, 24576, 17): 251.1, (4, 24763, 0): 266.2, (18, 24576, 17): 356.2, (18, 24763, 0): 357.9,
        (19, 24576, 17): 314.5, (19, 24763, 0): 319.1, (20, 24576, 17): 276.1, (20, 24763, 0): 279.9, (22, 23840, 20): 273.8,
        (22, 24763, 0): 271.4, (23, 24576, 17): 261.4, (23, 24763, 0): 269.5, (24, 23744, 20): 260.1, (24, 24763, 0): 264.1},
    (6171, 24576, 4096, SWIGLU): {(4, 6144, 13): 904.8, (4, 6171, 0): 951.3, (18, 6144, 13): 1245.9, (18, 6171, 0): 1266.1,
        (19, 6144, 13): 1108.0, (19, 6171, 0): 1122.4, (20, 6144, 13): 1006.1, (20, 6171, 0): 1023.8, (22, 5920, 20): 983.4,
        (22, 6171, 0): 989.1, (23, 6144, 13): 947.9, (23, 6171, 0): 972.4, (24, 5824, 23): 954.1, (24, 6171, 0): 961.9},
    (47176, 2560, 4096, RESIDUAL): {(4, 45824, 18): 857.3, (4, 47176, 0): 912.1, (18, 45824, 18): 1143.7,
        (18, 47176, 0): 1121.1, (19, 45824, 18): 1018.9, (19, 47176, 0): 1022.6, (20, 45824, 18): 995.5, (20, 47176, 0): 998.3,
        (22, 44960, 20): 958.1, (22, 47176, 0): 951.9, (23, 44160, 20): 912.5, (23, 47176, 0): 919.8, (24, 45696, 18): 914.8,
        (24, 47176, 0): 962.9},
    (29476, 4096, 12288, RESIDUAL): {(4, 28672, 18): 2210.3, (4, 29476, 0): 2313.3, (18, 28672, 18): 3075.7,
        (18, 29476, 0): 3032.6, (19, 28672, 18): 2683.4, (19, 29476, 0): 2720.4, (20, 28672, 18): 2554.5,
        (20, 29476, 0): 2591.5, (22, 28160, 20): 2477.2, (22, 29476, 0): 2475.4, (23, 27648, 20): 2359.5,
        (23, 29476, 0): 2389.9, (24, 28672, 18): 2361.1, (24, 29476, 0): 2440.7},
    (117949, 1024, 3072, RESIDUAL): {(4, 114688, 18): 690.6, (4, 117949, 0): 729.4, (18, 114688, 18): 972.6,
        (18, 117949, 0): 958.3, (19, 114688, 18): 828.3, (19, 117949, 0): 831.6, (20, 114688, 18): 843.6,
        (20, 117949, 0): 848.4, (22, 112640, 20): 774.3, (22, 117949, 0): 766.2, (23, 110592, 20): 733.5,
        (23, 117949, 0): 742.2, (24, 114688, 18): 730.1, (24, 117949, 0): 762.2},
}


@pytest.mark.parametrize("product", sorted(MANY_ROUNDS))
def test_the_last_of_many_rounds_is_counted(plan, product):
    rc, (v1, _, _, m1, v2, _, _) = plan(*product)
    assert rc == 0
    assert MANY_ROUNDS[product][v1, m1, v2] <= 1.01 * min(MANY_ROUNDS[product].values())


def test_weights_beyond_the_cache_are_not_read_twice(plan):
    for m, k in ((300, 4096), (1300, 1024)):
        assert plan(m, 151936, k, STORE_F32)[1][3] == m


# the same for fewer than 2048 columns, all rows in one tile
NARROW = {
    (8700, 1024, 1024, SWIGLU): {4: 24.9, 16: 29.8, 17: 27.4, 18: 30.0, 19: 33.5, 20: 29.1, 22: 19.6, 23: 21.3, 24: 23.8},
    (6000, 1536, 2048, SWIGLU): {4: 46.3, 16: 55.0, 17: 50.2, 18: 53.8, 19: 60.3, 20: 50.8, 22: 35.7, 23: 39.2, 24: 43.1},
    (8700, 1024, 4096, STORE): {4: 82.5, 16: 105.2, 17: 94.7, 18: 93.0, 19: 107.0, 20: 93.9, 22: 65.9, 23: 71.3, 24: 79.1},
    (8700, 1024, 2048, QKV_ROPE): {4: 51.3, 17: 53.4, 18: 56.4, 19: 63.4, 20: 70.9, 23: 43.2},
    (16500, 1280, 4096, QKV_ROPE): {4: 183.5, 17: 215.6, 18: 205.5, 19: 192.8, 20: 194.6, 23: 157.1},
}


@pytest.mark.parametrize("product", sorted(NARROW))
def test_narrow_products_get_a_tile_near_the_best_measured_one(plan, product):
    rc, (v1, _, _, m1, _, _, _) = plan(*product)
    assert rc == 0 and m1 == product[0]
    assert NARROW[product][v1] <= 1.05 * min(NARROW[product].values())


# the same for products that consume or prepare a folded norm
FOLDED = {
    (3000, 4096, 12288, RESIDUAL_NORM): {1: 365.5, 3: 317.0},
    (4400, 4096, 4096, RESIDUAL_NORM): {1: 267.2, 3: 185.2},
    (9000, 1024, 3072, RESIDUAL_NORM): {1: 107.1, 3: 95.5},
    (1000, 2560, 9728, RESIDUAL_NORM): {1: 270.0, 3: 110.2},
    (16500, 2560, 9728, RESIDUAL_NORM): {1: 881.9, 3: 822.6},
    (24000, 1024, 256, QKV_ROPE): {3: 33.1, 4: 40.0},
    (2200, 24576, 4096, SWIGLU): {2: 544.5, 3: 437.6, 4: 424.3},
    (9000, 6144, 1024, SWIGLU): {2: 155.1, 3: 126.4, 4: 121.1},
    (9000, 4096, 1024, QKV_ROPE): {3: 106.2, 4: 112.5},
}


@pytest.mark.parametrize("product", sorted(FOLDED))
def test_folded_norms_get_a_tile_near_the_best_measured_one(plan, product):
    v = binding.load_library().radix_debug_gemm_plan_folded(*product)
    assert FOLDED[product][v] <= 1.05 * min(FOLDED[product].values())


def test_folded_plan_rejects_what_no_tile_runs(plan):
    lib = binding.load_library()
    assert lib.radix_debug_gemm_plan_folded(0, 256, 64, STORE) == -2
    for nout, epilogue in ((128, QKV_ROPE), (384, RESIDUAL_NORM), (64, STORE), (256, RESIDUAL), (256, STORE_F32)):
        assert lib.radix_debug_gemm_plan_folded(8, nout, 64, epilogue) == -3, (nout, epilogue)
