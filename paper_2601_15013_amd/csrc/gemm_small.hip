// 16-bit MFMA GEMM for launches that the large tiles of gemm_mfma.hip leave much of the chip idle on:
// C[M, Nout] = A[M, K] * W[Nout, K]^T with the same fused epilogues, in tiles of 32x16 to 256x128.
//
// What bounds these launches is latency: a few dozen to a few thousand rows against a weight matrix that has to
// come from HBM once.  A 128-row tile gives such a launch 8 to 100 workgroups of 256 CUs, each of which walks all
// of K alone.  Splitting K over workgroups would shorten the walk, but an output element must be summed in the
// same order whatever M is (a row of the deduplicated and of the plain pass agree bit for bit), so the tiles get
// smaller instead: every element is the chain of matrix instructions of the large kernel with the same epilogue expressions,
// and the results are identical.
//
// Structure: k-tiles of 64 (a row is one 128-byte line) travel global -> LDS by global_load_lds_dwordx4 through a
// ring of NS stages; the fragments of the next tile (small wavefront blocks) or k-step (large ones) are read ahead of
// the MFMAs, so neither the LDS latency nor, with NS - 1 tiles in flight, that of the memory is on the MFMA chain.  One
// barrier per k-tile.  What is left per k-tile is the issue of the loads, about 40 cycles each in the wavefront that
// issues it: the smallest tiles spread them over the most CUs (32x16 with two wavefronts: three loads each).  The
// epilogue goes through LDS as fp32, from where every thread takes whole 16-byte pieces of a row.
//
// us per launch, fp16, best 128-row tile of gemm_mfma.hip -> this kernel, in a loop over one product whose weights come from
// HBM (the same launches inside a forward of one prompt, by the kernel trace: q|k|v 26.4 -> 10.8, mean of O and down
// 22.2 -> 7.0, gate/up 12.1 -> 7.3):
//   M 21:   N 4096 K 1024 (q|k|v) 21.6 -> 7.1, N 1024 K 2048 14.0 -> 5.4, N 6144 K 1024 (gate/up) 11.0 -> 6.2,
//           N 1024 K 3072 19.4 -> 6.8, N 4096 K 12288 96 -> 25
//   M 1072: N 1024 K 2048 19.7 -> 13.8, N 1024 K 3072 27.3 -> 18.7, N 4096 K 12288 169 -> 141
//   M 768:  N 24576 K 4096 183 -> 163, N 4096 K 12288 131 -> 112
// The 128x128 tile has four stages: with three, two tiles of 0.44 us each were in flight, less than the latency of weights that
// come from HBM (M 658: N 4096 K 12288 99.5 -> 89.6 us, N 4096 K 4096 35.9 -> 32.8, N 24576 K 4096 171 -> 166; five are no better).
#include <type_traits>

#include "gemm_async.h"
#include "kernels.h"

namespace {

template <int DT, int BM, int BN, int WAVES_M, int WAVES_N, int NS, int EPI>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_small_kernel(
    const typename Op<DT>::T* __restrict__ A, const typename Op<DT>::T* __restrict__ W, int M, int Nout, int K,
    void* __restrict__ out_, int tiles_m, int tiles_n, int band, int w_k, QkvEpilogue qe,
    ARowMap amap) {
    typedef typename Op<DT>::T T;
    typedef typename Op<DT>::V8 V8;
    constexpr int NW = WAVES_M * WAVES_N, NT = 64 * NW;
    constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
    constexpr int MB = WTM / 16, NB = WTN / 16;
    constexpr int A_LOADS = BM / (8 * NW), B_LOADS = BN / (8 * NW), LOADS = A_LOADS + B_LOADS;   // 1 KB wave-loads
    static_assert(A_LOADS * 8 * NW == BM && B_LOADS * 8 * NW == BN, "every wavefront issues the same number of loads");
    static_assert((NS - 1) * LOADS < 64, "vmcnt range");
    constexpr uint32_t STAGE_B = (BM + BN) * GEMM_BK * 2;
    constexpr bool SWIGLU = EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_SPLIT;
    constexpr bool ROPE = EPI == EPI_QKV_ROPE || EPI == EPI_QKV_ROPE_SPLIT;
    constexpr int PARTS = (EPI == EPI_SWIGLU_SPLIT || EPI == EPI_QKV_ROPE_SPLIT) ? 2 : 1;
    static_assert(!SWIGLU || BN % 64 == 0, "gate and up blocks come in pairs of 32 columns");
    static_assert(!ROPE || (BN % 128 == 0 && BM % 32 == 0 && NW <= 8), "Q/K-norm + RoPE epilogue: whole heads, whole blocks of 32 rows");
    constexpr int CP = BN + 4;                                  // fp32 tile pitch (floats)
    constexpr int HP = 128 + 8;                                  // 16-bit staging pitch (elements), ROPE only
    // the epilogue takes EROWS rows of the tile at a time: all of them, or what one row of wavefronts holds
    constexpr uint32_t EALL = BM * CP * 4 + (ROPE ? BM * HP * 2 : 0);
    constexpr int EROWS = EALL <= 72 * 1024 || EALL <= NS * STAGE_B ? BM : WTM;
    constexpr uint32_t EPI_B = EROWS * CP * 4 + (ROPE ? EROWS * HP * 2 : 0);
    constexpr uint32_t LDS_B = NS * STAGE_B > EPI_B ? NS * STAGE_B : EPI_B;
    __shared__ __attribute__((aligned(16))) char lds_all[LDS_B];

    const GemmTile tile = gemm_tile_of((int)blockIdx.x, tiles_m, tiles_n, band);
    const int m0 = tile.tm * BM, n0 = tile.tn * BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int r = lane & 15, g = lane >> 4;                     // operand row and k-group of a 16x16 block

    // ---- global loads: wave-load j of this wavefront fills tile rows [8 (wave + NW j), +8): lane L -> row + L / 8,
    // LDS chunk L % 8, global chunk (L % 8) ^ swizzle.  Rows past M repeat row M - 1; a row map as in gemm_mfma.hip.
    const int lrow = lane >> 3, lpc = lane & 7;
    const int m_last = M - 1 - m0;
    uint32_t a_off[A_LOADS], w_off[B_LOADS];
#pragma unroll
    for (int j = 0; j < A_LOADS; ++j) {
        const int row = 8 * (wave + NW * j) + lrow;
        int src = row < m_last ? row : m_last;
        if (amap.rows != nullptr) {
            const int m = m0 + src;
            src = m < amap.n_valid ? amap.rows[m] : 0;
            if (src < 0 || src >= amap.n_src) {
                set_status(amap.status, RADIX_ERR_BAD_TOKEN);
                src = src < 0 ? 0 : amap.n_src - 1;
            }
        }
        a_off[j] = (uint32_t)(((size_t)src * K + 8 * (lpc ^ gemm_swz(row))) * sizeof(T));
    }
#pragma unroll
    for (int j = 0; j < B_LOADS; ++j) {
        const int row = 8 * (wave + NW * j) + lrow;
        w_off[j] = (uint32_t)(((size_t)row * w_k + 8 * (lpc ^ gemm_swz(row))) * sizeof(T));
    }
    const char* a_base = (const char*)(A + (amap.rows != nullptr ? (size_t)0 : (size_t)m0 * K));
    const char* w_base = (const char*)(W + (size_t)n0 * w_k);
    const int KT = K / GEMM_BK, WKT = w_k / GEMM_BK;
    const uint32_t lds_base = lds_addr(lds_all);

    // EPI_QKV_ROPE: blocks of 16 rows of one head that a wavefront rotates at a time; where that is one in all, its rows'
    // positions are fetched here and the table rows behind the loop, so that neither is waited for at the end
    constexpr int RB = (EROWS / 16 + NW - 1) / NW;
    constexpr bool ROPE_EARLY = ROPE && RB == 1 && EROWS == BM && BN == 128 && PARTS == 1;
    int rope_pos = 0;
    RopeRow tab;
    RopeGain gains;
    if (ROPE_EARLY) {
        const int gm = m0 + 16 * wave + r;
        rope_pos = qe.pos_c[gm < M ? gm : M - 1];
    }
    // EPI_RESIDUAL: this thread's pieces of the residual tile are requested ahead of everything else
    constexpr int RES_IT = EROWS * BN / 4 / NT;
    constexpr bool RES_EARLY = EPI == EPI_RESIDUAL && EROWS == BM && RES_IT <= 8;
    f32x4 res[RES_IT];
    if (RES_EARLY) {
#pragma unroll
        for (int it = 0; it < RES_IT; ++it) {
            const int idx = tid + it * NT, row = idx / (BN / 4), c = 4 * (idx % (BN / 4));
            const int gm = m0 + row < M ? m0 + row : M - 1;
            res[it] = *reinterpret_cast<const f32x4*>((const float*)out_ + (size_t)gm * Nout + n0 + c);
        }
    }
    // the next tile to be loaded: its operands and how many weight tiles are left before they start over
    const char* a_ptr = a_base;
    const char* w_ptr = w_base;
    int w_left = WKT;
    // its loads that go with k-step `part` (half of them; part < 0: all)
    auto issue = [&](uint32_t so, int part) {
#pragma unroll
        for (int f = 0; f < LOADS; ++f) {
            if (part >= 0 && f * 2 / LOADS != part) continue;
            if (f < B_LOADS) dma16(w_ptr, w_off[f < B_LOADS ? f : 0], lds_base + so + BM * 128 + 1024 * (wave + NW * f));
            else dma16(a_ptr, a_off[f < B_LOADS ? 0 : f - B_LOADS], lds_base + so + 1024 * (wave + NW * (f - B_LOADS)));
        }
        if (part == 0) return;
        a_ptr += GEMM_BK * sizeof(T);
        w_ptr += GEMM_BK * sizeof(T);
        if (--w_left == 0) { w_left = WKT; w_ptr = w_base; }
    };
    uint32_t rd[2];                                             // k-step ks: chunk 4 ks + g of row r
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) rd[ks] = (uint32_t)(r * 128 + (((4 * ks + g) ^ gemm_swz(r)) << 4));
    const uint32_t a_rd = (uint32_t)(wm * WTM) * 128u, b_rd = (uint32_t)(BM + wn * WTN) * 128u;
    auto read_frags = [&](uint32_t so, int ks, V8 (&fa)[2][MB], V8 (&fb)[2][NB]) {
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            uint4 v = *reinterpret_cast<const uint4*>(lds_all + so + a_rd + rd[ks] + i * 2048);
            fa[ks][i] = *reinterpret_cast<V8*>(&v);
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            uint4 v = *reinterpret_cast<const uint4*>(lds_all + so + b_rd + rd[ks] + j * 2048);
            fb[ks][j] = *reinterpret_cast<V8*>(&v);
        }
    };
    f32x4 acc[NB][MB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[j][i][e] = 0.f;

    const int pre = KT < NS ? KT : NS;
    for (int t = 0; t < pre; ++t) issue((uint32_t)t * STAGE_B, -1);
    if (KT >= NS) wait_vmcnt_and_lds<(NS - 1) * LOADS>(); else wait_vmcnt_and_lds<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    uint32_t so = 0;                                            // stage of tile kt
    if constexpr (MB * NB >= 16) {
    // Large wavefront blocks: one register set per k-step, the barrier in the middle of a tile.  The 16 or more MFMAs of
    // a k-step cover the LDS latency of the reads for the next one.
    V8 fa[2][MB], fb[2][NB];
    read_frags(0, 0, fa, fb);
    auto mfmas = [&](int ks) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int i = 0; i < MB; ++i) acc[j][i] = Op<DT>::mfma16(fb[ks][j], fa[ks][i], acc[j][i]);
    };
    auto tile_step = [&](auto more_c) {
        constexpr bool MORE = decltype(more_c)::value;
        read_frags(so, 1, fa, fb);
        mfmas(0);
        __builtin_amdgcn_sched_barrier(0);
        wait_vmcnt_and_lds<MORE ? (NS - 2) * LOADS : 0>();      // tile kt + 1 is here, tile kt is read out
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const uint32_t so_n = so + STAGE_B == NS * STAGE_B ? 0u : so + STAGE_B;
        read_frags(so_n, 0, fa, fb);
        if (MORE) issue(so, -1);
        mfmas(1);
        __builtin_amdgcn_sched_barrier(0);
        so = so_n;
    };
    int kt = 0;
    for (; kt + NS < KT; ++kt) tile_step(std::true_type());
    for (; kt < KT; ++kt) tile_step(std::false_type());
    } else {
    V8 fa0[2][MB], fb0[2][NB], fa1[2][MB], fb1[2][NB];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) read_frags(0, ks, fa0, fb0);
    // Tile kt: its fragments are in fa / fb (requested one tile ago; returned once lgkmcnt is 0, so after the barrier
    // its stage is free in every wavefront and tile kt + NS goes there).  Reads, MFMAs and loads are dealt out over
    // the two k-steps (the scheduling barriers pin that order).
    // MORE: tile kt + NS exists; else every load left is waited for (the last NS tiles, on their way for long).
    auto step = [&](auto more_c, V8 (&fa)[2][MB], V8 (&fb)[2][NB], V8 (&fa_n)[2][MB], V8 (&fb_n)[2][NB]) {
        constexpr bool MORE = decltype(more_c)::value;
        wait_vmcnt_and_lds<MORE ? (NS - 2) * LOADS : 0>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const uint32_t so_n = so + STAGE_B == NS * STAGE_B ? 0u : so + STAGE_B;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            read_frags(so_n, ks, fa_n, fb_n);                   // past the last tile: a stage's old bytes, never used
            if (MORE) issue(so, ks);
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int i = 0; i < MB; ++i) acc[j][i] = Op<DT>::mfma16(fb[ks][j], fa[ks][i], acc[j][i]);
            __builtin_amdgcn_sched_barrier(0);
        }
        so = so_n;
    };
    int kt = 0;
    for (; kt + 1 + NS < KT; kt += 2) {
        step(std::true_type(), fa0, fb0, fa1, fb1);
        step(std::true_type(), fa1, fb1, fa0, fb0);
    }
    if (kt + NS < KT) {                                         // an odd tile that still has one to load; back to set 0
        step(std::true_type(), fa0, fb0, fa1, fb1);
        ++kt;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int i = 0; i < MB; ++i) fa0[ks][i] = fa1[ks][i];
#pragma unroll
            for (int j = 0; j < NB; ++j) fb0[ks][j] = fb1[ks][j];
        }
    }
    for (; kt + 1 < KT; kt += 2) {
        step(std::false_type(), fa0, fb0, fa1, fb1);
        step(std::false_type(), fa1, fb1, fa0, fb0);
    }
    if (kt < KT) step(std::false_type(), fa0, fb0, fa1, fb1);
    }

    // ---- epilogue: every load has landed (the last steps waited for all of them).  EROWS rows of the accumulators at a
    // time go to LDS, once the wavefronts are done with what was there: register e of acc[j][i] is row 16 i + r,
    // column 16 j + 4 g + e of this wavefront's block.
    float* const ct = reinterpret_cast<float*>(lds_all);
    asm volatile("" : "+v"(rope_pos));                          // nothing that needs it is computed, and so waited for, above the loop
    if (ROPE_EARLY && wave < EROWS / 16 && (n0 >> 7) < qe.n_q_heads + qe.n_kv_heads) {
        rope_load(tab, qe, rope_pos, g);
        rope_gain(gains, qe, (n0 >> 7) >= qe.n_q_heads, g);
    }
    T* const outp = (T*)out_;
    const int out_w = SWIGLU ? (Nout >> 1) : Nout, ldo = out_w * PARTS;
    const int ncol0 = SWIGLU ? (n0 >> 1) : n0;
    for (int pass = 0; pass < BM / EROWS; ++pass) {
    const int e0 = m0 + pass * EROWS;                           // first row of the pass
    __syncthreads();
    if (EPI == EPI_RESIDUAL && !RES_EARLY) {
#pragma unroll
        for (int it = 0; it < RES_IT; ++it) {
            const int idx = tid + it * NT, row = idx / (BN / 4), c = 4 * (idx % (BN / 4));
            const int gm = e0 + row < M ? e0 + row : M - 1;
            res[it] = *reinterpret_cast<const f32x4*>((const float*)out_ + (size_t)gm * Nout + n0 + c);
        }
    }
    if (EROWS == BM || wm == pass) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
                *reinterpret_cast<f32x4*>(ct + ((EROWS == BM ? wm * WTM : 0) + 16 * i + r) * CP + wn * WTN + 16 * j + 4 * g) = acc[j][i];
    }
    __syncthreads();

    if (EPI == EPI_RESIDUAL || EPI == EPI_STORE_F32) {
#pragma unroll
        for (int it = 0; it < RES_IT; ++it) {
            const int idx = tid + it * NT, row = idx / (BN / 4), c = 4 * (idx % (BN / 4));
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (EPI == EPI_RESIDUAL) v = res[it];
            const f32x4 p = *reinterpret_cast<const f32x4*>(ct + row * CP + c);
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] += p[t];
            if (e0 + row < M) *reinterpret_cast<f32x4*>((float*)out_ + (size_t)(e0 + row) * Nout + n0 + c) = v;
        }
        continue;
    }
    // 16-bit outputs, the heads of a q | k | v tile one after the other
#pragma unroll
    for (int hh = 0; hh < (ROPE ? BN / 128 : 1); ++hh) {
    const int head = (n0 >> 7) + hh;
    if (!ROPE || head >= qe.n_q_heads + qe.n_kv_heads) {
        constexpr int CHUNKS = (SWIGLU ? BN / 2 : (ROPE ? 128 : BN)) / 8;      // 16-byte pieces of an output row
        for (int idx = tid; idx < EROWS * CHUNKS; idx += NT) {
            const int row = idx / CHUNKS, c = 8 * (idx % CHUNKS) + 128 * hh;
            const float* p = ct + row * CP + (SWIGLU ? 2 * (c & ~31) + (c & 31) : c);
            T hi[8], lo[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                float y = p[t];
                if (SWIGLU) {
                    const float gt = y, up = p[t + 32];
                    // silu(g) * u with the hardware reciprocal (1 ulp) instead of an IEEE division
                    y = gt * __builtin_amdgcn_rcpf(1.0f + __expf(-gt)) * up;
                }
                hi[t] = (T)y;
                lo[t] = (T)(y - (float)hi[t]);
            }
            if (e0 + row < M) {
                T* o = outp + (size_t)(e0 + row) * ldo + ncol0 + c;
                *reinterpret_cast<uint4*>(o) = *reinterpret_cast<uint4*>(hi);
                if (PARTS == 2) *reinterpret_cast<uint4*>(o + out_w) = *reinterpret_cast<uint4*>(lo);
            }
        }
        continue;
    }
    if constexpr (ROPE) {
        // One q or k head: blocks of 16 rows are shared out over the wavefronts, and a lane takes the piece of a row that the
        // large kernel's accumulators would give it, so that the results are the same.
        T* const ht = reinterpret_cast<T*>(lds_all + EROWS * CP * 4);
        for (int part = 0; part < PARTS; ++part) {
            if (part || hh) __syncthreads();                    // the staging rows have been read
#pragma unroll
            for (int q = 0; q < RB; ++q) {
                const int ib = wave + NW * q;
                if (ib >= EROWS / 16) continue;
                if (!ROPE_EARLY) {
                    const int gm = e0 + 16 * ib + r;
                    rope_load(tab, qe, qe.pos_c[gm < M ? gm : M - 1], g);
                    rope_gain(gains, qe, head >= qe.n_q_heads, g);
                }
                const float* rowp = ct + (16 * ib + r) * CP + 128 * hh + 4 * g;
                f32x4 v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const f32x4*>(rowp + 16 * j);
                rope_apply([&](int j, int e) { return v[j][e]; }, tab, gains, qe, [&](int j, f32x4 y) {
                    T o[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        o[t] = (T)y[t];
                        if (part) o[t] = (T)(y[t] - (float)o[t]);
                    }
                    *reinterpret_cast<uint2*>(ht + (16 * ib + r) * HP + 16 * j + 4 * g) = *reinterpret_cast<uint2*>(o);
                });
            }
            __syncthreads();
            for (int idx = tid; idx < EROWS * 16; idx += NT) {
                const int row = idx >> 4, c = 8 * (idx & 15);
                if (e0 + row < M)
                    *reinterpret_cast<uint4*>(outp + (size_t)(e0 + row) * ldo + part * out_w + n0 + 128 * hh + c) =
                        *reinterpret_cast<const uint4*>(ht + row * HP + c);
            }
        }
    }
    }
    }
}

template <int DT, int BM, int BN, int WAVES_M, int WAVES_N, int NS>
int launch_small_cfg(const void* A, const void* W, int M, int Nout, int K, int w_k, int epilogue, void* out,
                     const QkvEpilogue& qe, const ARowMap& amap, hipStream_t stream) {
    typedef typename Op<DT>::T T;
    if (Nout % BN != 0 || K % GEMM_BK != 0 || w_k % GEMM_BK != 0) return RADIX_ERR_UNSUPPORTED;
    const int tiles_m = ceil_div(M, BM), tiles_n = Nout / BN;
    if ((long long)tiles_m * tiles_n > 0x7FFFFFFFLL) return RADIX_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)(tiles_m * tiles_n)), block(64 * WAVES_M * WAVES_N);
    // Few rows: all row tiles of a column tile are neighbours on one XCD, so that a weight strip enters one L2 only.
    // More rows than an L2 keeps: bands, as in the large kernel.
    const int band = (size_t)M * K * sizeof(T) <= (size_t)8 << 20 ? tiles_m : gemm_band_rows(BM, K, (int)sizeof(T), tiles_n);
#define RADIX_LAUNCH(E)                                                                                          \
    hipLaunchKernelGGL((gemm_small_kernel<DT, BM, BN, WAVES_M, WAVES_N, NS, E>), grid, block, 0, stream,         \
                       (const T*)A, (const T*)W, M, Nout, K, out, tiles_m, tiles_n, band, w_k, qe, amap)
    constexpr bool ALL = BM < 256;          // 256x128: heads and fp32 rows only (small_256x128), the others in gemm_mfma.hip
    switch (epilogue) {
        case EPI_STORE:
            if constexpr (ALL) { RADIX_LAUNCH(EPI_STORE); return RADIX_OK; }
            break;
        case EPI_RESIDUAL: RADIX_LAUNCH(EPI_RESIDUAL); return RADIX_OK;
        case EPI_STORE_F32: RADIX_LAUNCH(EPI_STORE_F32); return RADIX_OK;
        case EPI_SWIGLU:
            if constexpr (ALL && BN % 64 == 0) { RADIX_LAUNCH(EPI_SWIGLU); return RADIX_OK; }
            break;
        case EPI_SWIGLU_SPLIT:
            if constexpr (ALL && BN % 64 == 0) { RADIX_LAUNCH(EPI_SWIGLU_SPLIT); return RADIX_OK; }
            break;
        case EPI_QKV_ROPE:
            if constexpr (BN % 128 == 0 && BM % 32 == 0) { RADIX_LAUNCH(EPI_QKV_ROPE); return RADIX_OK; }
            break;
        case EPI_QKV_ROPE_SPLIT:
            if constexpr (BN % 128 == 0 && BM % 32 == 0) { RADIX_LAUNCH(EPI_QKV_ROPE_SPLIT); return RADIX_OK; }
            break;
        default: break;
    }
#undef RADIX_LAUNCH
    return RADIX_ERR_UNSUPPORTED;
}

template <int DT>
int launch_small_dt(int variant, const void* A, const void* W, int M, int Nout, int K, int w_k, int epilogue, void* out,
                    const QkvEpilogue& qe, const ARowMap& amap, hipStream_t s) {
    switch (variant) {
        case 11: return launch_small_cfg<DT, 32, 16, 2, 1, 8>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, s);
        case 12: return launch_small_cfg<DT, 32, 32, 2, 2, 8>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, s);
        case 13: return launch_small_cfg<DT, 32, 128, 1, 4, 4>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, s);
        case 14: return launch_small_cfg<DT, 32, 64, 2, 2, 6>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, s);
        case 15: return launch_small_cfg<DT, 64, 32, 2, 2, 5>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, s);
        case 16: return launch_small_cfg<DT, 64, 64, 2, 2, 4>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, s);
        case 17: return launch_small_cfg<DT, 64, 128, 2, 4, 3>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, s);
        case 18: return launch_small_cfg<DT, 128, 128, 2, 4, 4>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, s);
        case 19: return launch_small_cfg<DT, 128, 256, 2, 4, 3>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, s);
        case 20: return launch_small_cfg<DT, 256, 128, 4, 2, 3>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, s);
        default: return RADIX_ERR_UNSUPPORTED;
    }
}

}  // namespace

int launch_gemm_small(const void* A, const void* W, int M, int Nout, int K, int epilogue, void* out, int op_dtype,
                      int variant, hipStream_t stream, const QkvEpilogue& qkv, int w_k, const ARowMap& a_rows) {
    if (op_dtype == RADIX_BF16) return launch_small_dt<RADIX_BF16>(variant, A, W, M, Nout, K, w_k, epilogue, out, qkv, a_rows, stream);
    if (op_dtype == RADIX_F16) return launch_small_dt<RADIX_F16>(variant, A, W, M, Nout, K, w_k, epilogue, out, qkv, a_rows, stream);
    return RADIX_ERR_UNSUPPORTED;
}
