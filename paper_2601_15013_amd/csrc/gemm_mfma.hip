// 16-bit MFMA GEMM  C[M, Nout] = A[M, K] * W[Nout, K]^T  (fp32 accumulate) with fused epilogues,
// for bf16 or fp16 operands.
//
// These are the position-wise contractions of the method - Q/K/V and O projections and the
// SwiGLU MLP (paper: Background Eq. 5; Algorithm 1 "QKVProj", "OProj", "MLP") - run on the
// compact row count M = N' (or M = N in the no-dedup baseline).  Both operands are K-contiguous
// ("NT" GEMM), which is exactly the per-lane operand layout of v_mfma_f32_16x16x32_{bf16,f16}:
// lane (r = lane % 16, g = lane / 16) supplies 8 consecutive k of row r for k-group g.
//
// What bounds it is chip power: with random operands the matrix pipe alone, fed from registers, holds 1.66 PFLOP/s with
// v_mfma_f32_32x32x16 and 1.91 with v_mfma_f32_16x16x32 (2.48 and 2.44 with all-zero operands: the clock falls with
// switching power, and the smaller instruction reads and writes half as many accumulators per product).  The same loads and
// LDS reads in a loop of 32x32x16 took 7119 us for M 44032, N 24576, K 4096 (1.25 PFLOP/s), this one takes 6250 to 6360
// (1.40); K 12288, N 4096: 3714 -> 3160.  Without its global loads the loop would take 5220 of 6550 us, without its LDS
// reads 6150 (zero operands: 4330 and 5210 of 4860).
//
// Structure
//   * Workgroup tile BM x BN, k-tile 64, 4 or 8 wavefronts (one or two per SIMD) in a WAVES_M x WAVES_N
//     grid; each wavefront owns (BM/WAVES_M) x (BN/WAVES_N) outputs as 16x16 MFMA accumulators.
//   * The product is formed transposed, C^T = W * A^T (weights are the MFMA "A" operand), so a
//     lane owns one output ROW and 4 consecutive columns per block: the fp32 epilogues
//     (residual read-modify-write, plain fp32 store) access 16 bytes per lane straight from that
//     layout, the 16-bit ones transpose through LDS and store whole 256-byte row segments.
//   * Global -> LDS goes through global_load_lds_dwordx4 (no VGPR staging): a wavefront fills
//     1 KB of LDS per instruction, lane L landing at byte 16 L; the XOR swizzle that keeps the
//     fragment reads bank-conflict free is therefore applied to the GLOBAL address each lane
//     fetches.  A k-tile row is a whole 128-byte line: loads alone, in this tile order, reach 22 to 24 TB/s that way
//     (14.7 in half lines, 18.6 with the two halves requested back to back).  The
//     load is issued from inline assembly: issued through the compiler builtin, the compiler's
//     wait-count pass makes every later LDS read wait for ALL loads in flight (it cannot prove
//     that the reads of one slot do not alias the fills of the others), which serialises the
//     pipeline.  The only vector-memory waits are the explicit ones in front of the barriers.
//   * LDS holds D + 1 k-tiles of A and D of W (256x256: 3 and 2 in all 160 KB), one barrier per k-tile; details at the loop.
//   * K is consumed in order and there is no split-K, so an output element is reduced in the
//     same order wherever its row sits in the matrix: the deduplicated and the no-dedup pass
//     give bit-identical rows.
//   * Ragged M: rows >= M are fetched from row M-1 and never stored.
//   * Workgroups are numbered so that the 8 XCDs (round-robin dispatch) each work on a compact
//     band of row tiles, sweeping the weight tiles in step with the other XCDs (details at the tile
//     assignment), which keeps an XCD's L2 on few A rows and the shared memory-side cache on few W rows.
#include <type_traits>

#include "gemm_async.h"
#include "kernels.h"

namespace {

template <int DT, int BM, int BN, int WAVES_M, int WAVES_N, int EPI, bool FOLD>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_mfma_kernel(const typename Op<DT>::T* __restrict__ A,
                                                                 const typename Op<DT>::T* __restrict__ W, int M,
                                                                 int Nout, int K, void* __restrict__ out_,
                                                                 int tiles_m, int tiles_n, int w_k,
                                                                 QkvEpilogue qe, ARowMap amap, NormFusion nf, int BAND) {
    typedef typename Op<DT>::T T;
    typedef typename Op<DT>::V8 V8;
    typedef typename Op<DT>::V4 V4;
    constexpr int NW = WAVES_M * WAVES_N;                      // wavefronts: 4 (one per SIMD) or 8 (two per SIMD)
    static_assert(NW == 4 || NW == 8, "4 or 8 wavefronts");
    constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
    constexpr int MB = WTM / 16, NB = WTN / 16;
    // 1 KB wave-loads per wavefront per k-tile; where the rows of A do not share out evenly the first wavefronts have one more
    constexpr int A_LOADS = (BM / 8 + NW - 1) / NW, A_REM = BM / 8 % NW, B_LOADS = BN / (8 * NW);
    static_assert(BM % 8 == 0 && BN % (8 * NW) == 0, "whole wave-loads");
    constexpr uint32_t A_SLOT = BM * GEMM_BK * 2, B_SLOT = BN * GEMM_BK * 2;
    constexpr bool SWIGLU = EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_SPLIT;
    constexpr bool ROPE = EPI == EPI_QKV_ROPE || EPI == EPI_QKV_ROPE_SPLIT;
    constexpr int PARTS = (EPI == EPI_SWIGLU_SPLIT || EPI == EPI_QKV_ROPE_SPLIT) ? 2 : 1;     // (hi, lo) halves of the output row
    static_assert(!SWIGLU || (NB % 4 == 0), "SwiGLU needs gate/up block pairs of 32 columns in one wavefront");
    static_assert(!ROPE || WTN == 128, "Q/K-norm + RoPE epilogue: one wavefront = one 128-wide head");
    static_assert(EPI != EPI_RESIDUAL_NORM || WTN == 128, "sum-of-squares slots are 128 columns = one wavefront");
    static_assert(WTM % 16 == 0 && (NB == 4 || NB == 8), "whole blocks, k-step slices");

    constexpr int EPI_PITCH = 272;                             // epilogue row pitch in bytes (256 + 16 pad)
    constexpr uint32_t EPI_B = NW * 64 * EPI_PITCH;            // 64 rows per wavefront
    // k-tiles from one's first load to its use: as many as LDS holds.  256x256: two, in all 160 KB of a CU
    constexpr int D = 5 * A_SLOT + 4 * B_SLOT <= 160 * 1024 ? 4 : 4 * A_SLOT + 3 * B_SLOT <= 160 * 1024 ? 3 : 2;
    constexpr uint32_t RING_B = (D + 1) * A_SLOT + D * B_SLOT;
    __shared__ __attribute__((aligned(16))) char lds_all[RING_B > EPI_B ? RING_B : EPI_B];

    // ---- tile assignment (gemm_tile_of: XCD-aware bands of row tiles sweeping the column tiles)
    const GemmTile tile = gemm_tile_of((int)blockIdx.x, tiles_m, tiles_n, BAND);
    const int tm = tile.tm, tn = tile.tn;
    const int m0 = tm * BM, n0 = tn * BN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int r = lane & 15, g = lane >> 4;                     // operand row and k-group of a 16x16 block

    // ---- global-load assignment.  Wave-load j of this wavefront fills tile rows
    // [8 (wave + NW j), +8): lane L -> row + L / 8, LDS chunk L % 8, global chunk (L % 8) ^ swizzle.
    // Addresses are (uniform 64-bit tile base, advanced per k-tile) + (per-lane 32-bit byte offset).
    // With a row map (amap.rows != nullptr) row m of the product is row amap.rows[m] of A: the gather in front
    // of the output projection rides in these offsets instead of being a copy kernel of its own.  Rows at or
    // past amap.n_valid (padding of a bucketed compact space) take source row 0; entries outside
    // [0, amap.n_src) are clamped and reported.
    const int lrow = lane >> 3, lpc = lane & 7;
    const int m_last = M - 1 - m0;                              // last valid row of this tile (ragged M)
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
    const bool a_extra = A_REM == 0 || wave < A_REM;            // this wavefront has A_LOADS of them, not one less
#pragma unroll
    for (int j = 0; j < B_LOADS; ++j) {
        const int row = 8 * (wave + NW * j) + lrow;
        w_off[j] = (uint32_t)(((size_t)row * w_k + 8 * (lpc ^ gemm_swz(row))) * sizeof(T));
    }
    const char* a_ptr = (const char*)(A + (amap.rows != nullptr ? (size_t)0 : (size_t)m0 * K));    // next k-tile of A to be loaded
    const char* const w_base = (const char*)(W + (size_t)n0 * w_k);
    const char* w_ptr = w_base;                                                                  // and of W
    const int KT = K / GEMM_BK, WKT = w_k / GEMM_BK;
    int w_left = WKT;               // k-tiles left in the weight rows; past them they start over (A = [hi | lo] mode)

    f32x4 acc[NB][MB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[j][i][e] = 0.f;

    // EPI_QKV_ROPE: position ids of this lane's rows, fetched before the main loop so that the RoPE
    // table rows can be addressed without a dependent load when the epilogue starts
    int rope_pos[MB];
    if (ROPE) {
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            int gm = m0 + wm * WTM + i * 16 + r;
            gm = gm < M ? gm : M - 1;
            rope_pos[i] = qe.pos_c[gm];
        }
    }

    // RMSNorm folded in (consumer side): the first sum-of-squares slots of every row this lane owns are
    // requested here, ahead of the first tile loads, and added up once those are under way; the row scales
    // then sit in MB registers through the main loop (the epilogue would otherwise start with a chain of
    // dependent loads per tile).
    constexpr bool CONSUMES_NORM = FOLD && (EPI == EPI_STORE || EPI == EPI_SWIGLU || EPI == EPI_QKV_ROPE);
    constexpr int SS_EARLY = 16 / MB;                           // float2 loads per row requested early
    float2 ssv[MB][SS_EARLY];
    const bool scale_rows = CONSUMES_NORM && nf.ss_in != nullptr;
    if (scale_rows) {
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            int gm = m0 + wm * WTM + i * 16 + r;
            gm = gm < M ? gm : M - 1;
            const float* sp = nf.ss_in + (size_t)gm * nf.n_slots_in;
#pragma unroll
            for (int u = 0; u < SS_EARLY; ++u)
                ssv[i][u] = 2 * u < nf.n_slots_in ? *reinterpret_cast<const float2*>(sp + 2 * u) : make_float2(0.f, 0.f);
        }
    }

    // ---- LDS: D + 1 slots for k-tiles of A, then D for k-tiles of W; tile t lives in A slot t % (D + 1), W slot t % D
    // (wave-uniform offsets that rotate as the loop advances).
    const uint32_t lds_base = lds_addr(lds_all);
    uint32_t rd[2];                                             // k-step ks: chunk 4 ks + g of row r
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) rd[ks] = (uint32_t)(r * 128 + (((4 * ks + g) ^ gemm_swz(r)) << 4));
    const char* const a_rd = lds_all + (wm * WTM) * 128;
    const char* const b_rd = lds_all + (D + 1) * A_SLOT + (wn * WTN) * 128;
    auto load_a = [&](uint32_t slot, int f) {
        if (A_REM == 0 || f < A_LOADS - 1 || a_extra) dma16(a_ptr, a_off[f], lds_base + slot + 1024 * (wave + NW * f));
        if (f == A_LOADS - 1) a_ptr += GEMM_BK * sizeof(T);
    };
    auto load_b = [&](uint32_t slot, int f) {
        dma16(w_ptr, w_off[f], lds_base + (D + 1) * A_SLOT + slot + 1024 * (wave + NW * f));
        if (f == B_LOADS - 1) {
            w_ptr += GEMM_BK * sizeof(T);
            if (--w_left == 0) { w_left = WKT; w_ptr = w_base; }
        }
    };
    V8 fa0[MB], fa1[MB], fb[NB];                                // A fragments of the two k-steps, W fragments of the running one
    auto read_a = [&](V8& f, uint32_t slot, int ks, int i) {
        uint4 v = *reinterpret_cast<const uint4*>(a_rd + slot + rd[ks] + i * 2048);
        f = *reinterpret_cast<V8*>(&v);
    };
    auto read_b = [&](uint32_t slot, int ks, int j) {
        uint4 v = *reinterpret_cast<const uint4*>(b_rd + slot + rd[ks] + j * 2048);
        fb[j] = *reinterpret_cast<V8*>(&v);
    };

    // row scales from the sums of squares: slots in increasing order (the early ones, then the rest); adding the
    // zeros that stand in for slots a narrow model does not have changes nothing
    float rsr[MB];
    auto row_scales = [&]() {
#pragma unroll
        for (int i = 0; i < MB; ++i) rsr[i] = 1.0f;
        if (scale_rows) {
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                float ssum = 0.f;
#pragma unroll
                for (int u = 0; u < SS_EARLY; ++u) { ssum += ssv[i][u].x; ssum += ssv[i][u].y; }
                if (nf.n_slots_in > 2 * SS_EARLY) {
                    int gm = m0 + wm * WTM + i * 16 + r;
                    gm = gm < M ? gm : M - 1;
                    const float* sp = nf.ss_in + (size_t)gm * nf.n_slots_in;
                    for (int k0 = 2 * SS_EARLY; k0 < nf.n_slots_in; k0 += 2 * SS_EARLY) {
                        float2 more[SS_EARLY];
#pragma unroll
                        for (int u = 0; u < SS_EARLY; ++u)
                            more[u] = k0 + 2 * u < nf.n_slots_in ? *reinterpret_cast<const float2*>(sp + k0 + 2 * u)
                                                                 : make_float2(0.f, 0.f);
#pragma unroll
                        for (int u = 0; u < SS_EARLY; ++u) { ssum += more[u].x; ssum += more[u].y; }
                    }
                }
                rsr[i] = 1.0f / sqrtf(ssum * nf.inv_d + nf.eps);
            }
        }
    };

    uint32_t a_cur = 0, a_nxt = A_SLOT, a_far = D * A_SLOT, b_cur = 0, b_nxt = B_SLOT;     // slots of tiles t, t+1 and (A) t+D
#pragma unroll
    for (int t = 0; t < D; ++t) {
        if (t >= KT) break;
#pragma unroll
        for (int f = 0; f < A_LOADS; ++f) load_a(t * A_SLOT, f);
#pragma unroll
        for (int f = 0; f < B_LOADS; ++f) load_b(t * B_SLOT, f);
    }
    if (KT < D) wait_vmcnt<0>();
    else if (a_extra) wait_vmcnt<(D - 1) * (A_LOADS + B_LOADS)>();
    else wait_vmcnt<(D - 1) * (A_LOADS + B_LOADS - 1)>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < MB; ++i) read_a(fa0[i], a_cur, 0, i);
#pragma unroll
    for (int j = 0; j < NB - 1; ++j) read_b(b_cur, 0, j);
    row_scales();

    // One k-tile = two k-steps of 32, each of NB slices (the scheduling barriers pin the order): slice j multiplies W
    // fragment j with the MB fragments of A.  W fragments are reloaded in place for the next k-step, one slice after
    // their use; A fragments alternate between two sets.  What is read from LDS in a slice is used NB - 1 slices later.
    // Global loads, two per slice: A of tile t+D from the start of the first k-step, into the slot of tile t-1; W of tile
    // t+D in the second, into the slot of tile t, right after the barrier that says that every wavefront has read tile t
    // and has tile t+1 in LDS (spread over the k-step they land too late for the next barrier: 2 to 4 % with zero operands).
    // Every other slice runs its blocks backwards, so that two MFMAs in a row always share an operand: less switching
    // (registers only: 1.99 -> 2.04 PFLOP/s).
    // MODE 2: tile t+D exists; 1: tile t+1 does; 0: the last tile.
    constexpr int BAR = NB >= 8 ? 2 : 1;                        // the barrier stands ahead of this slice
    auto k_tile = [&](auto mode_c) {
        constexpr int MODE = decltype(mode_c)::value;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if (MODE == 2) {
#pragma unroll
                for (int f = 0; f < A_LOADS; ++f)
                    if (f / 2 == j) load_a(a_far, f);
            }
            if (j == 0) read_b(b_cur, 0, NB - 1);
            else read_b(b_cur, 1, j - 1);
#pragma unroll
            for (int i = 0; i < MB; ++i)
                if (1 + i * (NB - 2) / MB == j) read_a(fa1[i], a_cur, 1, i);
#pragma unroll
            for (int u = 0; u < MB; ++u) {
                const int i = j & 1 ? MB - 1 - u : u;
                acc[j][i] = Op<DT>::mfma16(fb[j], fa0[i], acc[j][i]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if (MODE > 0 && j == BAR) {
                if (MODE != 2) wait_vmcnt_and_lds<0>();
                else if (a_extra) wait_vmcnt_and_lds<(D - 1) * A_LOADS + (D - 2) * B_LOADS>();
                else wait_vmcnt_and_lds<(D - 1) * (A_LOADS - 1) + (D - 2) * B_LOADS>();
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            if (MODE == 2 && j >= BAR) {
#pragma unroll
                for (int f = 0; f < B_LOADS; ++f)
                    if (BAR + f / 2 == j) load_b(b_cur, f);
            }
            if (j == 0) read_b(b_cur, 1, NB - 1);
            if (MODE > 0 && j >= BAR) {
                if (j == BAR) {
#pragma unroll
                    for (int u = 0; u < BAR; ++u) read_b(b_nxt, 0, u);
                } else {
                    read_b(b_nxt, 0, j - 1);
                }
#pragma unroll
                for (int i = 0; i < MB; ++i)
                    if (BAR + i * (NB - BAR) / MB == j) read_a(fa0[i], a_nxt, 0, i);
            }
#pragma unroll
            for (int u = 0; u < MB; ++u) {
                const int i = j & 1 ? MB - 1 - u : u;
                acc[j][i] = Op<DT>::mfma16(fb[j], fa1[i], acc[j][i]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (D == 2) {
            const uint32_t a_t = a_cur, b_t = b_cur;
            a_cur = a_nxt; a_nxt = a_far; a_far = a_t;
            b_cur = b_nxt; b_nxt = b_t;
        } else {
            a_far = a_cur;
            a_cur = a_nxt; a_nxt = a_nxt == D * A_SLOT ? 0u : a_nxt + A_SLOT;
            b_cur = b_nxt; b_nxt = b_nxt == (D - 1) * B_SLOT ? 0u : b_nxt + B_SLOT;
        }
    };
    int t = 0;
    for (; t + D < KT; ++t) k_tile(std::integral_constant<int, 2>());
    if (D == 2) {
        if (KT > 1) k_tile(std::integral_constant<int, 1>());
    } else {
        for (; t + 1 < KT; ++t) k_tile(std::integral_constant<int, 1>());
    }
    k_tile(std::integral_constant<int, 0>());
    __builtin_amdgcn_s_barrier();     // every load has landed (the last waits were for all of them); wait until every
                                      // wavefront is done with the slots
    asm volatile("" ::: "memory");

    // ---- epilogue.  acc[j][i] register e holds output row 16 i + r, column 16 j + 4 g + e
    // of this wavefront's block: a lane owns a ROW.  To write full 128-byte lines the block goes
    // through LDS in passes of 64 rows: every lane drops its row pieces into a padded row-major
    // buffer private to its wavefront (row pitch 272 bytes), then the wavefront reads the buffer back
    // 16 bytes per lane, 16 lanes per 256-byte row, and does the global access from that layout.
    constexpr int PITCH = EPI_PITCH;
    char* const ebuf = lds_all + wave * (64 * PITCH);

    // The epilogue derives all its addresses from a lane id the compiler cannot see through, so that
    // none of that arithmetic is hoisted above the main loop, where every vector register counts.
    int lane_opaque = lane;
    asm volatile("" : "+v"(lane_opaque));
    {
    const int lane = lane_opaque;
    const int r = lane & 15, g = lane >> 4;

    if (CONSUMES_NORM) {            // in place: scaled as they are used, they would be held twice
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[j][i][e] *= rsr[i];
    }

    if (EPI == EPI_RESIDUAL_NORM) {
        // fp32 read-modify-write of the residual stream as below, plus, per row: the updated values times the
        // gain of the norm that follows, in the operand type (what the next projection multiplies), and the
        // sum of their squares over this wavefront's 128 columns (in-lane in column order, then the three other
        // lanes of the row).  The loads of a row block are all issued before
        // anything of the block before it is stored: written in that order by hand, because with three
        // unrelated pointers in play the compiler may not move a load above a store on its own, and every
        // (load, add, store) step would then pay the memory latency in turn.
        const int slot = (n0 + wn * WTN) >> 7, n_slots = Nout >> 7;
        const float* grow = nf.gain + n0 + wn * WTN;
        f32x4 gn[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) gn[j] = *reinterpret_cast<const f32x4*>(grow + 16 * j + 4 * g);
        f32x4 cur[NB], nxt[NB];
        auto load_block = [&](int i, f32x4* v) {
            const int gm = m0 + wm * WTM + i * 16 + r;
            const float* orow = (const float*)out_ + (size_t)(gm < M ? gm : M - 1) * Nout + n0 + wn * WTN;
#pragma unroll
            for (int j = 0; j < NB; ++j) v[j] = *reinterpret_cast<const f32x4*>(orow + 16 * j + 4 * g);
        };
        load_block(0, cur);
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            if (i + 1 < MB) load_block(i + 1 < MB ? i + 1 : 0, nxt);
            const int gm = m0 + wm * WTM + i * 16 + r;
            const bool live = gm < M;                              // all lanes of a row agree
            float* orow = (float*)out_ + (size_t)(live ? gm : M - 1) * Nout + n0 + wn * WTN;
            T* arow = (T*)nf.a16 + (size_t)(live ? gm : M - 1) * Nout + n0 + wn * WTN;
            float ss = 0.f;
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int c = 16 * j + 4 * g;
                f32x4 v = cur[j];
                V4 a;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    v[t] += acc[j][i][t];
                    ss += v[t] * v[t];
                    a[t] = (T)(v[t] * gn[j][t]);
                }
                if (live) {
                    *reinterpret_cast<f32x4*>(orow + c) = v;
                    *reinterpret_cast<V4*>(arow + c) = a;
                }
            }
            ss += __shfl_xor(ss, 16, 64);
            ss += __shfl_xor(ss, 32, 64);
            if (live && g == 0) nf.ss_out[(size_t)gm * n_slots + slot] = ss;
#pragma unroll
            for (int j = 0; j < NB; ++j) cur[j] = nxt[j];
        }
    } else if (EPI == EPI_RESIDUAL || EPI == EPI_STORE_F32) {
        // fp32 read-modify-write of the residual stream (or a plain fp32 store) straight from the accumulator layout: per
        // instruction 16 rows x 64 contiguous bytes; the loads of two row blocks are issued before their
        // stores, and nothing has to be converted, so the LDS detour does not pay here.
#pragma unroll
        for (int ip = 0; ip < MB; ip += 2) {
            constexpr int PAIR = 2;
            f32x4 v[PAIR][NB];
            float* orow[PAIR];
#pragma unroll
            for (int il = 0; il < PAIR; ++il) {
                if (ip + il >= MB) continue;
                const int gm = m0 + wm * WTM + (ip + il) * 16 + r;
                orow[il] = (float*)out_ + (size_t)(gm < M ? gm : M - 1) * Nout + n0 + wn * WTN + 4 * g;
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    v[il][j] = {0.f, 0.f, 0.f, 0.f};
                    if (EPI == EPI_RESIDUAL) v[il][j] = *reinterpret_cast<const f32x4*>(orow[il] + 16 * j);
                }
            }
#pragma unroll
            for (int il = 0; il < PAIR; ++il) {
                const int gm = m0 + wm * WTM + (ip + il) * 16 + r;
                if (ip + il >= MB || gm >= M) continue;
#pragma unroll
                for (int j = 0; j < NB; ++j) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) v[il][j][t] += acc[j][ip + il < MB ? ip + il : 0][t];
                    *reinterpret_cast<f32x4*>(orow[il] + 16 * j) = v[il][j];
                }
            }
        }
    } else {
        // 16-bit outputs.  EPI_STORE: 128 output columns per wavefront row (256 bytes);
        // EPI_SWIGLU: gate blocks j, j+1 and up blocks j+2, j+3 -> 64 output columns per row (128 bytes);
        // EPI_SWIGLU_SPLIT: the same twice, the rounded value into the left half of the output row and what
        // the rounding dropped into the right half (the down projection then runs over the doubled K).
        constexpr int OUT_COLS = SWIGLU ? WTN / 2 : WTN;
        constexpr int CHUNKS = OUT_COLS / 8;                    // 16-byte chunks per output row
        constexpr int ROWS_PER_INST = 64 / CHUNKS;
        const int orow = lane / CHUNKS, ochunk = lane % CHUNKS;
        const int out_w = SWIGLU ? (Nout >> 1) : Nout;          // logical output width; a (hi, lo) row is twice that
        const int ldo = out_w * PARTS;
        const int ncol0 = SWIGLU ? ((n0 + wn * WTN) >> 1) : (n0 + wn * WTN);
        // Q/K-norm + RoPE: which head this wavefront's columns are, and whether it is rotated (q, k) or not (v)
        const int head = (n0 + wn * WTN) >> 7;
        const bool rope_head = ROPE && head < qe.n_q_heads + qe.n_kv_heads;
        RopeGain gains;
        constexpr int TABS = PARTS == 2 || FOLD ? 1 : 2;        // two do not fit the registers of those epilogues
        RopeRow tab[TABS];
        // 256x256 with a folded norm: fetched once, the gains were more registers than there are (four accumulators spilled)
        constexpr bool GAINS_LATE = FOLD && MB * NB >= 32;
        if (rope_head && !GAINS_LATE) rope_gain(gains, qe, head >= qe.n_q_heads, g);
#pragma unroll
        for (int ip = 0; ip < MB; ip += 4) {
#pragma unroll
          for (int part = 0; part < PARTS; ++part) {
            if (TABS == 2 && rope_head) rope_load(tab[0], qe, rope_pos[ip], g);
#pragma unroll
            for (int il = 0; il < 4; ++il) {
                if (ip + il >= MB) continue;
                const int i = ip + il < MB ? ip + il : 0;
                char* rowp = ebuf + (il * 16 + r) * PITCH;
                if (SWIGLU) {
#pragma unroll
                    for (int j = 0; j < NB; ++j) {
                        if (j & 2) continue;                       // an up block
                        V4 v;
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const float gt = acc[j][i][t], up = acc[j + 2 < NB ? j + 2 : 0][i][t];
                            // silu(g) * u with the hardware reciprocal (1 ulp) instead of an IEEE division
                            const float y = gt * __builtin_amdgcn_rcpf(1.0f + __expf(-gt)) * up;
                            const T hi = (T)y;
                            v[t] = part == 0 ? hi : (T)(y - (float)hi);
                        }
                        *reinterpret_cast<V4*>(rowp + (((j >> 2) * 2 + (j & 1)) * 16 + 4 * g) * 2) = v;
                    }
                } else if (ROPE && rope_head) {
                    // This wavefront's 128 columns are exactly one q or k head of the fused q|k|v row.  The table rows of the
                    // next 16 rows are on their way while these are rotated: with the rows fetched as they are used, and the
                    // gains with them, this epilogue cost as much as 6 k-tiles more (M 8192, N 4096, K 1024: 84 -> 75 us a
                    // launch, 50432 rows 483 -> 444).
                    if (GAINS_LATE) rope_gain(gains, qe, head >= qe.n_q_heads, g);
                    if (TABS == 1) rope_load(tab[0], qe, rope_pos[i], g);
                    else if (il < 3 && i + 1 < MB) rope_load(tab[(il + 1) % TABS], qe, rope_pos[i + 1 < MB ? i + 1 : 0], g);
                    __builtin_amdgcn_sched_barrier(0);
                    rope_apply([&](int j, int e) { return acc[j < NB ? j : 0][i][e]; }, tab[il % TABS], gains, qe, [&](int j, f32x4 y) {
                        V4 v;
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const T hi = (T)y[t];
                            v[t] = part == 0 ? hi : (T)(y[t] - (float)hi);
                        }
                        *reinterpret_cast<V4*>(rowp + (16 * j + 4 * g) * 2) = v;
                    });
                    __builtin_amdgcn_sched_barrier(0);
                } else {
#pragma unroll
                    for (int j = 0; j < NB; ++j) {
                        V4 v;
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const float y = acc[j][i][t];
                            const T hi = (T)y;
                            v[t] = part == 0 ? hi : (T)(y - (float)hi);
                        }
                        *reinterpret_cast<V4*>(rowp + (16 * j + 4 * g) * 2) = v;
                    }
                }
            }
#pragma unroll
            for (int t = 0; t < (MB - ip < 4 ? (MB - ip) * 16 : 64) / ROWS_PER_INST; ++t) {
                const int row = orow + ROWS_PER_INST * t;
                const int gm = m0 + wm * WTM + ip * 16 + row;
                const uint4 v = *reinterpret_cast<const uint4*>(ebuf + row * PITCH + ochunk * 16);
                if (gm < M)
                    *reinterpret_cast<uint4*>((T*)out_ + (size_t)gm * ldo + part * out_w + ncol0 + ochunk * 8) = v;
            }
          }
        }
    }
    }
}

template <int DT, int BM, int BN, int WAVES_M, int WAVES_N>
int launch_cfg(const void* A, const void* W, int M, int Nout, int K, int w_k, int epilogue, void* out,
               const QkvEpilogue& qe, const ARowMap& amap, const NormFusion& nf, hipStream_t stream) {
    typedef typename Op<DT>::T T;
    if (Nout % BN != 0 || K % GEMM_BK != 0) return RADIX_ERR_UNSUPPORTED;
    const int tiles_m = ceil_div(M, BM), tiles_n = Nout / BN;
    dim3 grid((unsigned)(tiles_m * tiles_n)), block(64 * WAVES_M * WAVES_N);
    const int band_cfg = gemm_band_rows(BM, K, (int)sizeof(T), tiles_n);
#define RADIX_LAUNCH(E, FOLD)                                                                                 \
    do {                                                                                                      \
        auto kfn = gemm_mfma_kernel<DT, BM, BN, WAVES_M, WAVES_N, E, FOLD>;                                   \
        hipLaunchKernelGGL(kfn, grid, block, 0, stream, (const T*)A, (const T*)W, M, Nout, K, out, tiles_m,   \
                           tiles_n, w_k, qe, amap, nf, band_cfg);                                             \
        return RADIX_OK;                                                                                      \
    } while (0)
    // PLAIN: products without a folded norm; FOLDED: those with one, consumed or (four wavefronts) prepared
    constexpr bool EIGHT = WAVES_M * WAVES_N == 8, ROPE = BN / WAVES_N == 128;
    constexpr bool PLAIN = EIGHT && BM > 128, FOLDED = BM == 128 || (BM == 256 && BN == 256);
    if constexpr (FOLDED) {
        if (nf.ss_in != nullptr) {
            if constexpr (EIGHT || BM == 128) {
                if (epilogue == EPI_STORE) RADIX_LAUNCH(EPI_STORE, true);
                if (epilogue == EPI_SWIGLU) RADIX_LAUNCH(EPI_SWIGLU, true);
                if constexpr (ROPE)
                    if (epilogue == EPI_QKV_ROPE) RADIX_LAUNCH(EPI_QKV_ROPE, true);
            }
            return RADIX_ERR_UNSUPPORTED;
        }
    }
    if constexpr (PLAIN) {
        if constexpr (!(ROPE && BM == 192)) {
        if (epilogue == EPI_STORE) RADIX_LAUNCH(EPI_STORE, false);
        if (epilogue == EPI_RESIDUAL) RADIX_LAUNCH(EPI_RESIDUAL, false);
        if (epilogue == EPI_SWIGLU) RADIX_LAUNCH(EPI_SWIGLU, false);
        if (epilogue == EPI_SWIGLU_SPLIT) RADIX_LAUNCH(EPI_SWIGLU_SPLIT, false);
        if constexpr (BN == 256)            // 256x128: gemm_small.hip
            if (epilogue == EPI_STORE_F32) RADIX_LAUNCH(EPI_STORE_F32, false);
        }
        if constexpr (ROPE) {
            if (epilogue == EPI_QKV_ROPE) RADIX_LAUNCH(EPI_QKV_ROPE, false);
            if (epilogue == EPI_QKV_ROPE_SPLIT) RADIX_LAUNCH(EPI_QKV_ROPE_SPLIT, false);
        }
    }
    if constexpr (FOLDED && ROPE && !PLAIN)
        if (epilogue == EPI_RESIDUAL_NORM) RADIX_LAUNCH(EPI_RESIDUAL_NORM, false);
#undef RADIX_LAUNCH
    return RADIX_ERR_UNSUPPORTED;
}

// CUs of the device (a partition has fewer than the chip's 256); 256 where there is no device to ask
int device_cus() {
    static int n_cu = 0;
    if (n_cu == 0) {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
            cus = 256;
        n_cu = cus;
    }
    return n_cu;
}

template <int DT>
int launch_dt(const void* A, const void* W, int M, int Nout, int K, int w_k, int epilogue, void* out, int variant,
              const QkvEpilogue& qe, const ARowMap& amap, const NormFusion& nf, hipStream_t stream) {
    const bool rope = epilogue == EPI_QKV_ROPE || epilogue == EPI_QKV_ROPE_SPLIT;
    if (variant == 20) return launch_cfg<DT, 256, 128, 4, 2>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, nf, stream);
    if (variant == 22) return launch_cfg<DT, 160, 256, 2, 4>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, nf, stream);
    if (variant == 23 && rope) return launch_cfg<DT, 192, 256, 4, 2>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, nf, stream);
    if (variant == 23) return launch_cfg<DT, 192, 256, 2, 4>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, nf, stream);
    if (variant == 24) return launch_cfg<DT, 224, 256, 2, 4>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, nf, stream);
    if (variant == 4 && Nout % 256 == 0) return launch_cfg<DT, 256, 256, 4, 2>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, nf, stream);
    if (variant == 1 && Nout % 256 == 0) return launch_cfg<DT, 256, 256, 2, 2>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, nf, stream);
    if (variant == 3 && Nout % 256 == 0) return launch_cfg<DT, 128, 256, 4, 2>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, nf, stream);
    if (variant == 2) return launch_cfg<DT, 128, 128, 4, 2>(A, W, M, Nout, K, w_k, epilogue, out, qe, amap, nf, stream);
    return RADIX_ERR_UNSUPPORTED;
}

// ---- tile choice.  Time of a launch with tile shape s, in microseconds: workgroups run `per_cu` at a time on each CU
// in rounds.  Where that is one, a round costs fixed_us + epi_us (first loads, epilogue, by what it writes: 16-bit rows, q|k|v
// heads, fp32 rows added to, fp32 rows written) and, per 64 columns of K, step_us + share_us times the share of the CUs that it
// occupies (the clock and the memory-side cache are shared by all).  Where several run on a CU, a round of n per CU costs fixed_us,
// n epi_us and, per 64 columns, step_us (what a k-tile takes when nothing else runs on the CU: a chain of latencies) or n share_us
// if that is more.
// A launch that does not fill its last round pays for it in full; where several workgroups run on a CU, only up to eight rounds.
// (One per CU: 12 products of the 0.6B, 4B and 8B shapes at 22 row counts, 5 to 22 rounds.  Counted like this, launches of 8 to 22
// rounds take 0.98 to 1.03 of the model's time on average, at every fill of the last round; with the rounds beyond eight counted
// in fractions, nearly empty last rounds took 1.04 to 1.08 of it.)
// The constants are least-squares fits of the logarithm to timed launches on MI355X (fp16 operands), in two sets because rows
// of A shorter than 1024 leave a launch mostly epilogue and start-up, which long rows say little about:
//   long_k, K >= 1024: 336 (product, row count) pairs of the four projections of the 0.6B, 4B and 8B shapes and four others
//     (K 1024 .. 12288), M 8 .. 50000, weights from HBM: within 3 % (large tiles) to 13 % (the smallest) of a launch; the tile
//     they pick takes 0.5 % longer than the best one (a tenth of them more than 1 %, the worst 23 %).  Written fp32 rows from
//     60 more (heads of 151936 columns, K 1024 .. 4096, and N 8192, M 8 .. 4500): 0.4 %, the worst 10 %.  They leave 256x128 tiles
//     through LDS (gemm_small.hip): 151936 columns, K 1024, M 1000: 421 us, straight from the accumulators 592.
//   short_k: 53 products of K 64 .. 768 at 23 and 25 row counts from 1 to 130000; not least squares alone, but the time lost by what
//     is picked and, less, the model's error for tiles within 1.4 of the best, which is 6 to 13 %.  The picked tile takes 0.5 %
//     longer than the best (a tenth of them more than 1.5 %, the worst 21 %), and on 732 pairs outside the fit 0.5 % (2.5 %, 12 %).  bf16
//     operands, which were not in the fit, gain as much over the plans before as fp16 ones (3.6 % over 562 launches).
// The 256x256 tile wins where it fills the chip; the tiles of 160, 192 and 224 rows where that leaves less of the last round
// empty: M 8300, N 1024: K 3072 70.1 / 57.3 us (256 / 160 rows), K 2048 54.4 / 43.0; M 5000, N 7168, K 5120: 338 / 294 (192 rows);
// M 16500, N 4096, K 768 114.6 / 105.7 (224 rows); 129 of the 336 pairs have one of the three as their best.  Their constants of long_k
// are 2 % above the fit: among many estimates one that is low by chance would win, and the older tiles are the safer choice.
struct TileCost { double launch_us, fixed_us, step_us, share_us, epi_us[4]; };
struct TileShape { int variant, bm, bn, per_cu; TileCost long_k, short_k; };
constexpr int LONG_K = 1024;
const TileShape tile_shapes[] = {
    { 4, 256, 256, 1, {1.95,  4.74, 0.776, 0.714, {0.37, 6.56, 12.93,  4.25}}, {2.27, 4.35, 0.883, 0.290, {1.80, 8.59, 14.65, 8.82}}},
    {11,  32,  16, 3, {2.00,  0.00, 0.113, 0.079, {0.62, 0.50,  0.00,  0.70}}, {1.46, 0.31, 0.038, 0.038, {0.57, 0.00, 0.78, 0.56}}},
    {12,  32,  32, 2, {1.74,  0.00, 0.130, 0.110, {0.51, 0.50,  0.00,  1.50}}, {1.04, 0.55, 0.133, 0.117, {0.36, 0.00, 0.34, 0.45}}},
    {13,  32, 128, 2, {1.74,  0.00, 0.339, 0.244, {0.99, 0.46,  0.00,  2.20}}, {1.51, 0.79, 0.018, 0.193, {0.36, 1.02, 0.92, 0.48}}},
    {14,  32,  64, 2, {1.61,  0.00, 0.191, 0.157, {1.89, 6.30,  0.00,  1.80}}, {1.45, 0.61, 0.009, 0.150, {0.14, 0.00, 0.54, 0.33}}},
    {15,  64,  32, 2, {1.09,  0.00, 0.183, 0.151, {1.00, 1.00,  0.17,  1.15}}, {1.24, 0.86, 0.024, 0.129, {0.27, 0.00, 0.38, 0.34}}},
    {16,  64,  64, 2, {3.13,  0.00, 0.084, 0.214, {0.17, 0.55,  0.00,  1.10}}, {1.27, 0.61, 0.015, 0.160, {0.69, 0.00, 1.18, 0.71}}},
    {17,  64, 128, 2, {1.88,  0.00, 0.443, 0.334, {0.36, 0.79,  0.00,  2.50}}, {1.31, 0.56, 0.017, 0.270, {0.93, 1.86, 1.40, 1.12}}},
    {18, 128, 128, 1, {1.75,  2.63, 0.367, 0.155, {0.48, 2.12,  1.46,  3.40}}, {0.20, 1.94, 0.172, 0.339, {1.45, 3.65, 3.96, 2.57}}},
    {19, 128, 256, 1, {3.29,  3.58, 0.598, 0.306, {0.10, 5.33,  2.45,  0.85}}, {2.19, 3.52, 0.099, 0.898, {0.04, 6.79, 4.96, 2.63}}},
    {20, 256, 128, 1, {2.40,  2.15, 0.551, 0.295, {0.34, 9.36,  6.02,  6.80}}, {0.50, 3.09, 0.385, 0.346, {0.68, 11.33, 6.35, 5.19}}},
    {22, 160, 256, 1, {3.44,  2.44, 0.663, 0.411, {0.33, 0.51,  6.95,  3.60}}, {0.70, 2.61, 0.460, 0.397, {1.72, 0.00, 9.98, 7.06}}},
    {23, 192, 256, 1, {2.42,  4.06, 0.731, 0.444, {0.00, 4.57,  9.41,  3.35}}, {1.03, 3.96, 0.589, 0.434, {0.66, 6.46, 11.11, 5.19}}},
    {24, 224, 256, 1, {3.16,  3.86, 0.799, 0.569, {0.24, 0.31, 10.22,  3.90}}, {1.82, 3.89, 0.581, 0.597, {1.13, 0.00, 12.52, 5.64}}},
};
double tile_time(const TileShape& sh, const TileCost& c, int cus, int M, int Nout, int K, int epilogue) {
    const double epi = c.epi_us[epilogue == EPI_QKV_ROPE || epilogue == EPI_QKV_ROPE_SPLIT ? 1 :
                                epilogue == EPI_RESIDUAL || epilogue == EPI_RESIDUAL_NORM ? 2 :
                                epilogue == EPI_STORE_F32 ? 3 : 0];
    const long long tiles = (long long)ceil_div(M, sh.bm) * (Nout / sh.bn);
    const double kt = K / 64;
    if (sh.per_cu == 1) {
        auto round_us = [&](double busy) { return c.fixed_us + epi + kt * (c.step_us + c.share_us * busy); };
        const int rest = (int)(tiles % cus);
        return c.launch_us + (double)(tiles / cus) * round_us(1.0) + (rest ? round_us((double)rest / cus) : 0.0);
    }
    double per = (double)tiles / cus;
    if (per < 8.0) per = (double)((tiles + cus - 1) / cus);
    const double full = (double)(long long)(per / sh.per_cu), rest = per - full * sh.per_cu;
    auto round_us = [&](double n) {
        return c.fixed_us + n * epi + kt * (n * c.share_us > c.step_us ? n * c.share_us : c.step_us);
    };
    return c.launch_us + full * round_us(sh.per_cu) + (rest > 0 ? round_us(rest) : 0.0);
}

double tile_time(const TileShape& sh, int cus, int M, int Nout, int K, int epilogue) {
    return tile_time(sh, K >= LONG_K ? sh.long_k : sh.short_k, cus, M, Nout, K, epilogue);
}

bool tile_usable(const TileShape& sh, int Nout, int epilogue) {
    if (Nout % sh.bn != 0) return false;
    if (epilogue == EPI_QKV_ROPE || epilogue == EPI_QKV_ROPE_SPLIT)                               // whole heads
        return sh.bn % 128 == 0 && sh.variant != 22 && sh.variant != 24;
    if (epilogue == EPI_SWIGLU || epilogue == EPI_SWIGLU_SPLIT) return sh.bn % 64 == 0;           // gate/up pairs
    return true;
}

// whole: only tiles that divide the rows
int best_tile(int cus, int M, int Nout, int K, int epilogue, bool whole, double* us) {
    int v = 0;
    for (const TileShape& sh : tile_shapes) {
        if (!tile_usable(sh, Nout, epilogue) || (whole && M % sh.bm != 0)) continue;
        const double t = tile_time(sh, cus, M, Nout, K, epilogue);
        if (v == 0 || t < *us) { *us = t; v = sh.variant; }
    }
    return v;
}

// Tiles of a product with a folded norm, in one launch.  Consumers run in eight wavefronts (two per SIMD, 256 registers each); the
// epilogue that prepares a norm holds a row block twice and needs a wavefront block 128 columns wide: four wavefronts of 512
// registers, or 128 rows.  Constants as above, K of any length, from 22 products (K 256 .. 12288, both kinds of epilogue) at 17 row
// counts from 20 to 44000: within 8 % of a launch, and the tile they pick takes 0.1 % longer than the best one (the worst 14 %).
const TileShape folded_shapes[] = {
    {4, 256, 256, 1, {1.59,  5.62, 0.974, 0.575, {0.82, 7.95, 0.00, 0.00}}, {}},
    {3, 128, 256, 1, {1.28,  2.94, 0.534, 0.357, {0.93, 4.31, 9.82, 0.00}}, {}},
    {2, 128, 128, 1, {1.28,  2.06, 0.309, 0.217, {0.81, 0.00, 0.00, 0.00}}, {}},
    {1, 256, 256, 1, {0.00, 18.36, 1.235, 0.721, {0.00, 0.00, 8.12, 0.00}}, {}},
};
int folded_tile(int cus, int M, int Nout, int K, int epilogue) {
    const bool prepares = epilogue == EPI_RESIDUAL_NORM, heads = epilogue == EPI_QKV_ROPE;
    int v = 0;
    double best = 0.0;
    for (const TileShape& sh : folded_shapes) {
        if (Nout % sh.bn != 0 || (prepares ? sh.variant == 4 : sh.variant == 1)) continue;
        if ((heads || prepares) && sh.bn != 256) continue;                       // wavefront blocks of 128 columns
        const double t = tile_time(sh, sh.long_k, cus, M, Nout, K, epilogue);
        if (v == 0 || t < best) { best = t; v = sh.variant; }
    }
    return v;
}

// Which loop a 256x128 tile runs: that of gemm_small.hip, whose epilogue goes through LDS, for heads, written fp32 rows and, where
// rows of A are short, rows added to - straight from the accumulators those cost as much as three to four k-tiles more.  us, large
// loop / this one: M 50000: N 640 K 640 74.8 / 71.8, N 640 K 1280 120.8 / 114.0; M 24000: N 384 K 384 28.3 / 24.6, N 1024 K 2048
// 106.8 / 108.7; M 130000 N 1024 K 3072 899 / 893, M 8200 78.0 / 83.3: from K 2048 on neither is better, from 3072 on the large one.
bool small_256x128(int K, int epilogue) {
    return epilogue == EPI_QKV_ROPE || epilogue == EPI_QKV_ROPE_SPLIT || epilogue == EPI_STORE_F32 || (epilogue == EPI_RESIDUAL && K < 2048);
}

// Tiles of a product: rows [0, m1) in tiles of shape v1, the rest (if any) in a second launch of shape v2.  The large
// tiles are at their best when the last round of workgroups is full; where M leaves a round nearly empty - 8240 rows
// are 33 row tiles of 256, and 32 of them are whole rounds of the chip - the rows past the last full round go to smaller
// tiles (M 8240, K 1024, N 4096: 111 us in one launch of 256x256, 93 us split; K 3072, N 1024: 79 and 62 us; with more rounds:
// M 16436, N 6144, K 2560 444 and 426, M 47176, N 2560, K 4096 912 and 857).
struct GemmPlan { int v1, m1, v2; };
GemmPlan plan_gemm(int cus, int M, int Nout, int K, int epilogue) {
    double whole = 0.0;
    GemmPlan p = {best_tile(cus, M, Nout, K, epilogue, false, &whole), M, 0};
    if (M <= 256 || K < 512) return p;
    // what a split has to beat: a launch more, and the model's own error, which is larger where K is short (N 2048: K 640, M 8200 39.6
    // whole, 36.2 split, and M 33000 110 and 113; below K 512 16 of 18 splits took longer than the best tile alone)
    double best = (K >= LONG_K ? 0.97 : 0.90) * whole;
    // weights too large for the memory-side cache come from HBM again in a second launch, which is as much as the last of many
    // rounds costs (300 and 1300 rows of a head of 151936 columns: 542 -> 614 and 570 -> 630 us)
    const bool weights_pass = (long long)Nout * K * 2 > 256LL << 20;
    for (const TileShape& sh : tile_shapes) {
        if (sh.bm < 128 || !tile_usable(sh, Nout, epilogue)) continue;
        const long long row_tiles = M / sh.bm, per_row = Nout / sh.bn;
        const long long rounds = row_tiles * per_row / cus;
        if (rounds < 1 || (rounds >= 8 && weights_pass)) continue;
        const long long m1 = rounds * cus / per_row * sh.bm;
        if (m1 < sh.bm || m1 >= M) continue;
        double t1 = 0.0, t2 = 0.0;              // rows that fill rounds of this tile may still run faster in another one
        const int v1 = best_tile(cus, (int)m1, Nout, K, epilogue, true, &t1);
        const int v2 = best_tile(cus, M - (int)m1, Nout, K, epilogue, false, &t2);
        if (t1 + t2 < best) { best = t1 + t2; p = {v1, (int)m1, v2}; }
    }
    return p;
}

}  // namespace

int launch_gemm_mfma(const void* A, const void* W, int M, int Nout, int K, int epilogue, void* out, int op_dtype,
                     int variant, hipStream_t stream, const QkvEpilogue* qkv, int w_k, const ARowMap* a_rows,
                     const NormFusion* norm) {
    if (M <= 0 || Nout <= 0) return RADIX_OK;
    if (K <= 0) return RADIX_ERR_UNSUPPORTED;
    if (w_k == 0) w_k = K;
    if (w_k != K && (2 * w_k != K || w_k % GEMM_BK != 0)) return RADIX_ERR_UNSUPPORTED;
    if ((((uintptr_t)A | (uintptr_t)W | (uintptr_t)out) & 15) != 0) return RADIX_ERR_MISALIGNED;
    QkvEpilogue qe = {};
    if (epilogue == EPI_QKV_ROPE || epilogue == EPI_QKV_ROPE_SPLIT) {
        if (!qkv || Nout % 256 != 0) return RADIX_ERR_UNSUPPORTED;
        qe = *qkv;
    }
    ARowMap amap = {};
    if (a_rows && a_rows->rows) {
        // per-lane 32-bit byte offsets now span the whole source matrix
        if (a_rows->n_src <= 0 || (long long)a_rows->n_src * K * 2 >= (1LL << 32)) return RADIX_ERR_UNSUPPORTED;
        amap = *a_rows;
    }
    NormFusion nf = {};
    if (norm) nf = *norm;
    if (epilogue == EPI_RESIDUAL_NORM) {
        if (Nout % 256 != 0 || !nf.a16 || !nf.gain || !nf.ss_out) return RADIX_ERR_UNSUPPORTED;
        if ((((uintptr_t)nf.a16 | (uintptr_t)nf.gain) & 15) != 0) return RADIX_ERR_MISALIGNED;
    }
    if (nf.ss_in && (nf.n_slots_in <= 0 || nf.n_slots_in % 2 != 0 || ((uintptr_t)nf.ss_in & 7) != 0)) return RADIX_ERR_UNSUPPORTED;
    const bool folded = nf.ss_in != nullptr || epilogue == EPI_RESIDUAL_NORM;
    if (folded && variant >= 11) return RADIX_ERR_UNSUPPORTED;
    auto launch = [&](int v, const void* a, int m, void* o) -> int {
        if ((v >= 11 && v < 20) || (v == 20 && small_256x128(K, epilogue))) return launch_gemm_small(a, W, m, Nout, K, epilogue, o, op_dtype, v, stream, qe, w_k, amap);
        if (op_dtype == RADIX_BF16) return launch_dt<RADIX_BF16>(a, W, m, Nout, K, w_k, epilogue, o, v, qe, amap, nf, stream);
        if (op_dtype == RADIX_F16) return launch_dt<RADIX_F16>(a, W, m, Nout, K, w_k, epilogue, o, v, qe, amap, nf, stream);
        return RADIX_ERR_UNSUPPORTED;
    };
    if (folded && variant == 0) variant = folded_tile(device_cus(), M, Nout, K, epilogue);
    if (folded || variant != 0) return launch(variant, A, M, out);
    if (K % GEMM_BK != 0) return RADIX_ERR_UNSUPPORTED;
    const GemmPlan plan = plan_gemm(device_cus(), M, Nout, K, epilogue);
    if (plan.v1 == 0) return RADIX_ERR_UNSUPPORTED;
    const int rc = launch(plan.v1, A, plan.m1, out);
    if (rc != RADIX_OK || plan.m1 == M) return rc;
    // the second launch sees the rows from m1 on
    size_t out_row = (size_t)Nout * 4;                             // EPI_RESIDUAL, EPI_STORE_F32, EPI_QKV_ROPE_SPLIT
    if (epilogue == EPI_STORE || epilogue == EPI_QKV_ROPE || epilogue == EPI_SWIGLU_SPLIT) out_row = (size_t)Nout * 2;
    else if (epilogue == EPI_SWIGLU) out_row = (size_t)Nout;
    if (qe.pos_c) qe.pos_c += plan.m1;
    const void* a2 = A;
    if (amap.rows) {
        amap.rows += plan.m1;
        amap.n_valid = amap.n_valid > plan.m1 ? amap.n_valid - plan.m1 : 0;
    } else {
        a2 = (const char*)A + (size_t)plan.m1 * K * 2;
    }
    return launch(plan.v2, a2, M - plan.m1, (char*)out + (size_t)plan.m1 * out_row);
}

// Host-side views of the tile numbering, for tests (declared in radixmlp_bench.h).
extern "C" int radix_debug_gemm_tile(int32_t bid, int32_t tiles_m, int32_t tiles_n, int32_t band, int32_t* tm, int32_t* tn) {
    if (!tm || !tn) return RADIX_ERR_NULL_POINTER;
    if (tiles_m <= 0 || tiles_n <= 0 || band <= 0 || bid < 0 || (long long)bid >= (long long)tiles_m * tiles_n) return RADIX_ERR_BAD_SIZE;
    const GemmTile t = gemm_tile_of(bid, tiles_m, tiles_n, band);
    *tm = t.tm;
    *tn = t.tn;
    return RADIX_OK;
}
extern "C" int radix_debug_gemm_band(int32_t tile_rows, int32_t K, int32_t tiles_n) {
    if (tile_rows <= 0 || K <= 0 || tiles_n <= 0) return RADIX_ERR_BAD_SIZE;
    return gemm_band_rows(tile_rows, K, 2, tiles_n);
}
extern "C" int radix_debug_gemm_plan_cus(int32_t cus, int32_t M, int32_t Nout, int32_t K, int32_t epilogue, int32_t* v1,
                                         int32_t* bm1, int32_t* bn1, int32_t* m1, int32_t* v2, int32_t* bm2, int32_t* bn2) {
    if (!v1 || !bm1 || !bn1 || !m1 || !v2 || !bm2 || !bn2) return RADIX_ERR_NULL_POINTER;
    if (cus <= 0 || M <= 0 || Nout <= 0 || K <= 0 || epilogue < 0) return RADIX_ERR_BAD_SIZE;
    const GemmPlan p = plan_gemm(cus, M, Nout, K, epilogue);
    *m1 = p.m1;
    *bm1 = *bn1 = *bm2 = *bn2 = 0;
    for (const TileShape& sh : tile_shapes) {
        if (sh.variant == p.v1) { *bm1 = sh.bm; *bn1 = sh.bn; }
        if (sh.variant == p.v2) { *bm2 = sh.bm; *bn2 = sh.bn; }
    }
    *v1 = p.v1;
    *v2 = p.v2;
    return p.v1 ? RADIX_OK : RADIX_ERR_UNSUPPORTED;
}
extern "C" int radix_debug_gemm_plan(int32_t M, int32_t Nout, int32_t K, int32_t epilogue, int32_t* v1, int32_t* bm1,
                                     int32_t* bn1, int32_t* m1, int32_t* v2, int32_t* bm2, int32_t* bn2) {
    return radix_debug_gemm_plan_cus(device_cus(), M, Nout, K, epilogue, v1, bm1, bn1, m1, v2, bm2, bn2);
}
extern "C" int radix_debug_gemm_plan_us(int32_t M, int32_t Nout, int32_t K, int32_t epilogue, int32_t v1, int32_t m1, int32_t v2,
                                        double* us) {
    if (!us) return RADIX_ERR_NULL_POINTER;
    if (M <= 0 || Nout <= 0 || K <= 0 || epilogue < 0 || m1 <= 0 || m1 > M) return RADIX_ERR_BAD_SIZE;
    double t1 = -1.0, t2 = -1.0;
    for (const TileShape& sh : tile_shapes) {
        if (!tile_usable(sh, Nout, epilogue)) continue;
        if (sh.variant == v1) t1 = tile_time(sh, device_cus(), m1, Nout, K, epilogue);
        if (m1 < M && sh.variant == v2) t2 = tile_time(sh, device_cus(), M - m1, Nout, K, epilogue);
    }
    if (t1 < 0.0 || (m1 < M && t2 < 0.0)) return RADIX_ERR_UNSUPPORTED;
    *us = m1 < M ? t1 + t2 : t1;
    return RADIX_OK;
}
extern "C" int radix_debug_gemm_plan_folded(int32_t M, int32_t Nout, int32_t K, int32_t epilogue) {
    if (M <= 0 || Nout <= 0 || K <= 0) return RADIX_ERR_BAD_SIZE;
    if (epilogue != EPI_STORE && epilogue != EPI_SWIGLU && epilogue != EPI_QKV_ROPE && epilogue != EPI_RESIDUAL_NORM) return RADIX_ERR_UNSUPPORTED;
    const int v = folded_tile(device_cus(), M, Nout, K, epilogue);
    return v ? v : RADIX_ERR_UNSUPPORTED;
}
// One product on the device with the tile named (0: what the plan picks), for tests that compare the tiles.
extern "C" int radix_debug_gemm_run(const void* A, const void* W, int32_t M, int32_t Nout, int32_t K, int32_t w_k, int32_t epilogue,
                                    void* out, int32_t op_dtype, int32_t variant, const float* gq, const float* gk,
                                    const float* cos_tab, const float* sin_tab, const int32_t* pos, int32_t n_q_heads,
                                    int32_t n_kv_heads, int32_t qk_norm, const int32_t* rows, int32_t n_valid, int32_t n_src,
                                    int32_t* status, void* stream) {
    if (!A || !W || !out) return RADIX_ERR_NULL_POINTER;
    if (M <= 0 || Nout <= 0 || K <= 0) return RADIX_ERR_BAD_SIZE;
    const bool rope = epilogue == EPI_QKV_ROPE || epilogue == EPI_QKV_ROPE_SPLIT;
    if (epilogue == EPI_RESIDUAL_NORM || epilogue < 0) return RADIX_ERR_UNSUPPORTED;
    if (rope && (!gq || !gk || !cos_tab || !sin_tab || !pos)) return RADIX_ERR_NULL_POINTER;
    if (rope && (n_q_heads < 0 || n_kv_heads < 0 || Nout != (n_q_heads + 2 * n_kv_heads) * 128)) return RADIX_ERR_BAD_SIZE;
    if (rows && (!status || n_valid < 0 || n_valid > M)) return RADIX_ERR_BAD_SIZE;
    if (variant != 0) {
        bool known = false;
        for (const TileShape& sh : tile_shapes)
            known = known || (sh.variant == variant && tile_usable(sh, Nout, epilogue));
        if (!known) return RADIX_ERR_UNSUPPORTED;
    }
    const QkvEpilogue qe = {gq, gk, cos_tab, sin_tab, pos, n_q_heads, n_kv_heads, qk_norm, 1e-6f};
    const ARowMap amap = {rows, n_valid, n_src, status};
    const int rc = launch_gemm_mfma(A, W, M, Nout, K, epilogue, out, op_dtype, variant, (hipStream_t)stream, rope ? &qe : nullptr,
                                    w_k, rows ? &amap : nullptr);
    if (rc != RADIX_OK) return rc;
    HIP_TRY(hipGetLastError());
    return RADIX_OK;
}
extern "C" int radix_debug_gemm_run_folded(const void* A, const void* W, int32_t M, int32_t Nout, int32_t K, int32_t epilogue,
                                           void* out, int32_t op_dtype, int32_t variant, const float* gq, const float* gk,
                                           const float* cos_tab, const float* sin_tab, const int32_t* pos, int32_t n_q_heads,
                                           int32_t n_kv_heads, const float* ss_in, int32_t n_slots_in, float inv_d, float eps,
                                           void* a16, const float* gain, float* ss_out, void* stream) {
    if (!A || !W || !out) return RADIX_ERR_NULL_POINTER;
    if (M <= 0 || Nout <= 0 || K <= 0) return RADIX_ERR_BAD_SIZE;
    if (variant < 0 || variant > 4) return RADIX_ERR_UNSUPPORTED;
    const bool rope = epilogue == EPI_QKV_ROPE, produces = epilogue == EPI_RESIDUAL_NORM;
    if (!rope && !produces && epilogue != EPI_STORE && epilogue != EPI_SWIGLU) return RADIX_ERR_UNSUPPORTED;
    if (produces ? !a16 || !gain || !ss_out : !ss_in) return RADIX_ERR_NULL_POINTER;
    if (rope && (!gq || !gk || !cos_tab || !sin_tab || !pos)) return RADIX_ERR_NULL_POINTER;
    if (rope && (n_q_heads < 0 || n_kv_heads < 0 || Nout != (n_q_heads + 2 * n_kv_heads) * 128)) return RADIX_ERR_BAD_SIZE;
    const QkvEpilogue qe = {gq, gk, cos_tab, sin_tab, pos, n_q_heads, n_kv_heads, 1, 1e-6f};
    const NormFusion nf = {a16, gain, ss_out, produces ? nullptr : ss_in, n_slots_in, inv_d, eps};
    const int rc = launch_gemm_mfma(A, W, M, Nout, K, epilogue, out, op_dtype, variant, (hipStream_t)stream, rope ? &qe : nullptr, K,
                                    nullptr, &nf);
    if (rc != RADIX_OK) return rc;
    HIP_TRY(hipGetLastError());
    return RADIX_OK;
}
