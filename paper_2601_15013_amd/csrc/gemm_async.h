// What the MFMA GEMM kernels share: asynchronous global -> LDS copies and the waits that go with them, the k-tile's layout in
// LDS, and the Q/K-norm + RoPE arithmetic of the q | k | v epilogue.
#pragma once
#include "common.h"
#include "kernels.h"

namespace {

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding: vmcnt = imm[15:14|3:0],
// expcnt = imm[6:4], lgkmcnt = imm[11:8]).
template <int N> __device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is 6 bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
// the same, and all LDS reads of this wavefront have returned (lgkmcnt = 0)
template <int N> __device__ __forceinline__ void wait_vmcnt_and_lds() {
    static_assert(N >= 0 && N < 64, "vmcnt is 6 bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (0 << 8));
}

// Asynchronous 16-byte-per-lane copy global -> LDS: lane L of the wavefront writes LDS bytes
// [lds_base + 16 L, +16).  lds_base must be wave-uniform.  (s_nop: M0 write -> LDS-DMA hazard.)
// The global address is (uniform 64-bit base) + (per-lane 32-bit byte offset).
__device__ __forceinline__ void dma16(const void* base, uint32_t lane_off, uint32_t lds_base) {
    // the base is wave-uniform by construction; readfirstlane states that where the compiler has parked it in
    // vector registers (it must reach the instruction in a scalar register pair)
    const uint64_t b = (uint64_t)(uintptr_t)base;
    // (the builtin returns a signed int: through uint32_t, or a low half with its top bit set would sign-extend
    // over the high half)
    const uint64_t bs = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32)) << 32) |
                        (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 ::"v"(lane_off), "s"(bs), "s"(lds_base) : "memory");
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p;
}

// k-tile of the GEMM kernels: 128 bytes = a whole cache line = 8 chunks of 16 bytes per operand row, in LDS too.
constexpr int GEMM_BK = 64;
// LDS chunk c of a tile row holds chunk c ^ gemm_swz(row): two rows span the 64 banks, so XORing the chunk index with bits
// 1..3 of the row sends 16 consecutive rows of one chunk column to 16 distinct 16-byte bank groups.
__device__ __forceinline__ int gemm_swz(int row) { return (row >> 1) & 7; }

// One quarter of a q or k head's row, as the accumulators of a 16-row block hold it: lane (r, g) has columns 16 j + 4 g + e of
// row r in v[j][e].  Paper: Q/K norms and RoPE are position-wise, hence run on compact rows ("Integration with Attention").
// The tables' pieces of the row and the gains' (columns 16 j + 4 g + e, j < 4):
struct RopeRow { f32x4 cs[4], sn[4]; };
struct RopeGain { f32x4 a[4], b[4]; };
__device__ __forceinline__ void rope_load(RopeRow& t, const QkvEpilogue& qe, int pos, int g) {
    const float* ct = qe.cos_tab + (size_t)pos * 64 + 4 * g;
    const float* st = qe.sin_tab + (size_t)pos * 64 + 4 * g;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        t.cs[j] = *reinterpret_cast<const f32x4*>(ct + 16 * j);
        t.sn[j] = *reinterpret_cast<const f32x4*>(st + 16 * j);
    }
}
__device__ __forceinline__ void rope_gain(RopeGain& t, const QkvEpilogue& qe, bool key_head, int g) {
    const float* gain = (key_head ? qe.gk : qe.gq) + 4 * g;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        t.a[j] = t.b[j] = f32x4{1.f, 1.f, 1.f, 1.f};
        if (qe.qk_norm) {
            t.a[j] = *reinterpret_cast<const f32x4*>(gain + 16 * j);
            t.b[j] = *reinterpret_cast<const f32x4*>(gain + 16 * j + 64);
        }
    }
}
// The per-head RMSNorm is an in-lane sum of 32 squares plus two exchanges; the rotary partner of column c < 64 (block j) is
// column c + 64 (block j + 4) of the same lane and register.  out(j, y): the four results of block j.
template <typename V, typename F>
__device__ __forceinline__ void rope_apply(const V& v, const RopeRow& t, const RopeGain& gn, const QkvEpilogue& qe, F out) {
    float rs = 1.0f;
    if (qe.qk_norm) {
        float ss = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) ss = __builtin_fmaf(v(j, e), v(j, e), ss);
        ss += __shfl_xor(ss, 16, 64);
        ss += __shfl_xor(ss, 32, 64);
        rs = 1.0f / sqrtf(ss * (1.0f / 128.0f) + qe.eps);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f32x4 ya, yb;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float xa = v(j, e) * rs * gn.a[j][e];
            const float xb = v(j + 4, e) * rs * gn.b[j][e];
            ya[e] = __builtin_fmaf(xa, t.cs[j][e], -(xb * t.sn[j][e]));
            yb[e] = __builtin_fmaf(xb, t.cs[j][e], xa * t.sn[j][e]);
        }
        out(j, ya);
        out(j + 4, yb);
    }
}

}  // namespace
