// Asynchronous global -> LDS copies and the waits that go with them, shared by the MFMA GEMM kernels.
#pragma once
#include "common.h"

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

}  // namespace
