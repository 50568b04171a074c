/*
 * radixmlp_bench.h - benchmark instrumentation of libradixmlp, kept apart from the product ABI
 * (radixmlp.h): per-kernel timing with HIP events on the caller's stream.
 */
#ifndef RADIXMLP_BENCH_H
#define RADIXMLP_BENCH_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Optional per-kernel timing for benchmarks.  While a category's bit is set in category_mask,
 * the forward calls bracket every every_nth-th launch of that category (0 or 1: every launch) with a
 * pair of HIP events recorded on the caller's stream; an event pair costs a few microseconds of idle
 * GPU around the launch it brackets, so timing inside a timed region should sample sparsely when
 * launches are short.  radix_timing_collect waits for the device, writes for every category the
 * summed elapsed milliseconds and the number of timed launches since the last collect/enable
 * (arrays of RADIX_TIMING_CATEGORIES entries, HOST pointers) and resets the counters.
 * Process-wide state, not thread-safe; meant for one benchmarking thread.  Mask 0 disables.
 */
enum {
    RADIX_TIME_GEMM_QKV = 0,
    RADIX_TIME_GEMM_O = 1,
    RADIX_TIME_GEMM_GATEUP = 2,
    RADIX_TIME_GEMM_DOWN = 3,
    RADIX_TIME_ATTENTION = 4,
    RADIX_TIME_SCATTER = 5,
    RADIX_TIME_GATHER = 6,
    RADIX_TIME_ROWOPS = 7,
    RADIX_TIME_GEMM_HILO = 8,      /* every GEMM of a layer that runs with (hi, lo) inputs (doubled K) */
    RADIX_TIMING_CATEGORIES = 9
};
int radix_timing_enable(uint32_t category_mask, uint32_t every_nth);
int radix_timing_collect(float* total_ms_host, int32_t* launches_host);

/*
 * Host-side views of the launch geometry, for tests (no GPU is touched).
 * radix_debug_gemm_tile: the output tile (*tm, *tn) that workgroup `bid` of a launch of tiles_m x tiles_n
 * workgroups computes when row tiles are grouped in bands of `band` - the same function the kernel calls.
 * radix_debug_gemm_band: the band width the launcher picks for 16-bit operands, row tiles of tile_rows rows and
 * rows of K elements (>= 1), or a negative status.
 * radix_debug_gemm_plan: the tiles a 16-bit product C[M, Nout] = A[M, K] W^T with epilogue code `epilogue` runs in: rows
 * [0, *m1) in tiles of shape *v1 (*bm1 x *bn1), the rest, if *m1 < M, in tiles of shape *v2 (*bm2 x *bn2).
 * Shapes: 4 is 256x256, 22 to 24 are 160, 192 and 224 rows of 256 columns, 20 is 256x128, 11 to 19 are the smaller ones.
 * radix_debug_gemm_plan_cus: the same for a device (a partition) of `cus` CUs instead of the present one.
 * radix_debug_gemm_plan_us: the time that the cost model behind that choice gives such a split (v2 is not read if m1 == M).
 * radix_debug_gemm_plan_folded: the tile of a product that consumes a folded norm (epilogue 0, 2 or 3) or prepares one (6): 1 and 4 are
 * 256x256 with four and eight wavefronts, 2 128x128, 3 128x256.  Or a negative status.
 * radix_debug_index_first_round: 1 if the index builder spreads its first round over the whole chip for B sequences of N
 * tokens together, 0 if one workgroup runs it, or a negative status.
 * radix_debug_index_host_slots: how many of the words of pinned memory through which radix_build_index answers are free (64 when
 * no call is running), 0 before the first call made them.
 */
int radix_debug_gemm_plan(int32_t M, int32_t Nout, int32_t K, int32_t epilogue, int32_t* v1, int32_t* bm1, int32_t* bn1,
                          int32_t* m1, int32_t* v2, int32_t* bm2, int32_t* bn2);
int radix_debug_gemm_plan_cus(int32_t cus, int32_t M, int32_t Nout, int32_t K, int32_t epilogue, int32_t* v1, int32_t* bm1,
                              int32_t* bn1, int32_t* m1, int32_t* v2, int32_t* bm2, int32_t* bn2);
int radix_debug_gemm_plan_us(int32_t M, int32_t Nout, int32_t K, int32_t epilogue, int32_t v1, int32_t m1, int32_t v2, double* us);
int radix_debug_gemm_plan_folded(int32_t M, int32_t Nout, int32_t K, int32_t epilogue);
int radix_debug_gemm_tile(int32_t bid, int32_t tiles_m, int32_t tiles_n, int32_t band, int32_t* tm, int32_t* tn);
int radix_debug_gemm_band(int32_t tile_rows, int32_t K, int32_t tiles_n);
int radix_debug_index_first_round(int32_t B, int32_t N);
int radix_debug_index_host_slots(void);

/*
 * One 16-bit product out = epilogue(A[M, K] W[Nout, w_k]^T) on the device in tiles of shape `variant` (as reported by
 * radix_debug_gemm_plan; 0: the tiles of the plan), for tests that compare the tiles with each other.  Device pointers,
 * caller-owned; out has the type and width of the epilogue.  Epilogue codes: 0 store, 1 add to fp32 rows, 2 SwiGLU, 3 q|k|v with
 * norm and RoPE, 4 store fp32, 5 and 7: 2 and 3 as (hi, lo) pairs.  w_k: K, or K / 2 for rows of A that are (hi, lo) pairs (0: K).
 * The q|k|v epilogues read gq, gk [128], cos, sin [positions, 64] and pos[M].  rows (may be NULL): row m < n_valid of the product is
 * row rows[m] of A's n_src rows, the others row 0; bad entries are clamped and reported in *status.
 */
int radix_debug_gemm_run(const void* A, const void* W, int32_t M, int32_t Nout, int32_t K, int32_t w_k, int32_t epilogue, void* out,
                         int32_t op_dtype, int32_t variant, const float* gq, const float* gk, const float* cos_tab,
                         const float* sin_tab, const int32_t* pos, int32_t n_q_heads, int32_t n_kv_heads, int32_t qk_norm,
                         const int32_t* rows, int32_t n_valid, int32_t n_src, int32_t* status, void* stream);

/*
 * The same with a folded RMSNorm (radix_model_config.fold_norms).  Epilogues 0, 2 and 3 consume one: rows are scaled by
 * 1 / sqrt(sum of the n_slots_in (even) values ss_in[m, :] * inv_d + eps) before the epilogue proper.  Epilogue 6 adds to the
 * fp32 rows of out and prepares one: a16[M, Nout] = rows * gain[Nout] in the operand type, ss_out[M, Nout / 128] = sums of squares of
 * 128 columns.  variant: 4 (256x256) and 2 (128x128, not for heads) consume, 1 (256x256) prepares, 3 (128x256) does both;
 * 0: the tile the launcher picks.
 */
int radix_debug_gemm_run_folded(const void* A, const void* W, int32_t M, int32_t Nout, int32_t K, int32_t epilogue, void* out,
                                int32_t op_dtype, int32_t variant, const float* gq, const float* gk, const float* cos_tab,
                                const float* sin_tab, const int32_t* pos, int32_t n_q_heads, int32_t n_kv_heads, const float* ss_in,
                                int32_t n_slots_in, float inv_d, float eps, void* a16, const float* gain, float* ss_out, void* stream);

#ifdef __cplusplus
}
#endif
#endif /* RADIXMLP_BENCH_H */
