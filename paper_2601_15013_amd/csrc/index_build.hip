// GPU builder of the prefix-trie index maps I_scatter / I_gather.
//
// What is computed is fixed by the paper (Approach, "Trie Construction" and "Gather and Scatter
// Kernels"; appendix Algorithm 2 with its "Index semantics"): nodes are path-specific, compact
// ids are handed out in order of first occurrence.  How it is computed here is not the
// sequential insertion of Algorithm 2 but a level-synchronous, "follow the leader" scheme:
//
//   * Every sequence s follows a leader: the lowest-numbered sequence known to share s's path
//     so far.  All sequences start by following the first non-empty sequence.
//   * One round = one trie branching level on each follower's path.  A wavefront compares the
//     follower with its leader 256 tokens (first round over the chip: 512) at a time (coalesced loads + ballot) until the first
//     (token, position) mismatch m.  Positions below m are duplicates of the leader's nodes.
//   * Followers that leave the same leader at the same depth with the same (token, position)
//     key enter the same child node.  They are grouped by an exact open-addressing table
//     (keys are compared in full, the hash only picks the probe start); the lowest-numbered
//     member becomes the leader of the new node and all its later positions are new nodes,
//     the others follow it in the next round.
//   * A sequence becomes a leader at most once, so there are at most (deepest branching
//     chain) rounds, and every position is compared exactly once: O(N) work in total.
//   * New nodes of sequence s are its positions >= b_s (the depth where it became a leader),
//     a contiguous tail, so compact ids are cbase_s + (p - b_s) with cbase the exclusive
//     wavefront scan of (len_s - b_s) over sequences: exactly first-occurrence order.
//
// The chain phase runs in one 1024-thread workgroup (it is latency-bound bookkeeping over B
// sequences), but for the comparisons of its first round in large batches; the final map write-out is a chip-wide
// kernel over tokens.
#include <mutex>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "radixmlp_bench.h"

namespace {

constexpr int IDX_THREADS = 1024;
constexpr int IDX_WAVES = IDX_THREADS / RADIX_WAVE;
constexpr int LCP_UNROLL = 4;
// sequences whose state (22 bytes each) and grouping table (two slots of 8 bytes each) are kept in LDS: 19 and 152 KB
constexpr int LDS_SEQ_FEW = 512, LDS_SEQ_MANY = 4096;

__device__ __forceinline__ int ld_agent(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// status word and N' for the host that waits for them (host: two words of its memory, or null)
__device__ __forceinline__ void tell_host(int32_t* host, int status, int n_compact) {
    if (!host) return;
    __hip_atomic_store(host, status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(host + 1, n_compact, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ uint32_t key_hash(int l, int m, int t, int pp) {
    uint64_t x = (((uint64_t)(uint32_t)l << 32) | (uint32_t)m) * 0x9E3779B97F4A7C15ull;
    x ^= ((uint64_t)(uint32_t)pp << 32) | (uint32_t)t;
    x ^= x >> 29;
    x *= 0xBF58476D1CE4E5B9ull;
    x ^= x >> 32;
    return (uint32_t)x;
}

// Comparison of follower s with its leader l from position st on, by one wavefront: the first position where they
// differ (or the shorter length); lead[] of the equal positions is written on the way, if given.
template <int UNROLL>
__device__ __forceinline__ int common_prefix(const int32_t* __restrict__ tok, const int32_t* __restrict__ pos, int bs,
                                             int bl, int st, int lim, int l, int32_t* __restrict__ lead, int lane) {
    for (int p0 = st; p0 < lim; p0 += 64 * UNROLL) {
        int neq[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            int p = p0 + u * 64 + lane;
            bool valid = p < lim;
            int a = valid ? tok[bs + p] : 0;
            int b = valid ? tok[bl + p] : 1;
            int d = (a != b);
            if (pos != nullptr && valid) d |= (pos[bs + p] != pos[bl + p]);
            neq[u] = d;
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            int p = p0 + u * 64 + lane;
            unsigned long long mask = __ballot(neq[u]);
            if (mask != 0ull) {
                int first = __ffsll((long long)mask) - 1;
                if (lead && lane < first) lead[bs + p] = l;
                return p0 + u * 64 + first;
            }
            if (lead) lead[bs + p] = l;
        }
    }
    return lim;
}

// Smallest s in [lo, hi] with cu[s + 1] > x, which holds at hi, by a wavefront: 64 candidates a step.  (A malformed cu gives
// some s of the range.)
__device__ __forceinline__ int first_end_behind(const int32_t* __restrict__ cu, int lo, int hi, int x, int lane) {
    while (lo < hi) {
        const int step = (hi - lo) / 64 + 1;                // candidates lo + step (lane + 1) - 1, the last one at or behind hi
        const int c = lo + step * (lane + 1) - 1;
        const unsigned long long behind = __ballot(cu[(c < hi ? c : hi) + 1] > x);
        if (behind == 0ull) break;
        const int f = __ffsll((long long)behind) - 1;       // the first candidate whose sequence ends behind x
        const int nh = lo + step * (f + 1) - 1;
        lo = lo + step * f;
        if (nh < hi) hi = nh;
    }
    return lo;
}

// Validation of cu_seqlens (before anything is dereferenced through it) and the initial state, by one workgroup.
// Returns the first non-empty sequence, which everybody else follows, or -1 on a malformed array.
// first: null, or what index_first_round_kernel found: where a follower leaves the first sequence.
template <int BATCH>
__device__ __forceinline__ int index_init(const int32_t* __restrict__ cu, int B, int N, int32_t* hdr, int32_t* ldr,
                                          int32_t* dep, int32_t* bdep, int32_t* mis, const int32_t* first, int32_t* n_compact_dev) {
    __shared__ int sh_first;
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid == 0) {
        hdr[0] = 0;             // every call starts with a clean status word
        sh_first = B;
    }
    // BATCH sequences per thread at a time, so that their loads are in flight together
    int c0[BATCH], c1[BATCH], f[BATCH];
    auto fetch = [&](int base) {
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int s = base + u * IDX_THREADS + tid;
            c0[u] = s < B ? cu[s] : 0;
            c1[u] = s < B ? cu[s + 1] : 0;
            f[u] = first != nullptr && s < B ? first[s] : -1;
        }
    };
    int bad = tid == 0 && (cu[0] != 0 || cu[B] != N);
    __syncthreads();
    for (int base = 0; base < B; base += BATCH * IDX_THREADS) {
        fetch(base);
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int s = base + u * IDX_THREADS + tid;
            if (c0[u] < 0 || c0[u] > N || c1[u] < c0[u] || c1[u] > N) bad = 1;
            const unsigned long long some = __ballot(c1[u] > c0[u]);
            if (lane == 0 && some != 0ull) atomicMin(&sh_first, s + __ffsll((long long)some) - 1);
        }
    }
    bad = __syncthreads_or(bad);
    if (bad) {
        if (tid == 0) {
            set_status(hdr, RADIX_ERR_BAD_CU_SEQLENS);
            hdr[1] = 0;
            *n_compact_dev = 0;
        }
        return -1;
    }
    const int s0 = sh_first;
    for (int base = 0; base < B; base += BATCH * IDX_THREADS) {
        if (B > BATCH * IDX_THREADS) fetch(base);
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int s = base + u * IDX_THREADS + tid, len = c1[u] - c0[u];
            if (s >= B) continue;
            if (len == 0 || s == s0) {
                bdep[s] = 0;      // leader from depth 0 (or empty)
                ldr[s] = -1;
                mis[s] = -1;
            } else {
                bdep[s] = f[u] == len ? len : -1;       // -1 marks an active follower; else (as in step 1 below) it ran out of tokens
                ldr[s] = f[u] == len ? -1 : s0;
                mis[s] = f[u] == len ? -1 : f[u];
                dep[s] = 0;
            }
        }
    }
    __syncthreads();
    return s0;
}

// Validation of cu_seqlens alone, in front of a first round that writes into I_scatter.
__global__ __launch_bounds__(IDX_THREADS) void index_check_kernel(const int32_t* __restrict__ cu, int B, int N, int32_t* hdr) {
    int bad = threadIdx.x == 0 && (cu[0] != 0 || cu[B] != N);
    for (int s = threadIdx.x; s < B; s += IDX_THREADS) {
        const int c0 = cu[s], c1 = cu[s + 1];
        if (c0 < 0 || c0 > N || c1 < c0 || c1 > N) bad = 1;
    }
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) hdr[0] = bad ? RADIX_ERR_BAD_CU_SEQLENS : 0;
}

// The comparisons of the first round, one wavefront per sequence over the whole chip: all sequences start by following
// the first non-empty one, so this is where the prefix that a batch shares is read, and most of what there is to compare.
// first[s]: where sequence s leaves it (its length, if it does not).  The chain kernel checks cu_seqlens and reports; here a
// malformed array must only do no harm: every sequence's own ends are checked before anything is read through them, and the maps
// are not written (lead null: the write-out takes the leader of the positions below first[s] from there).  With lead, the
// leaders are written and index_check_kernel ran before (checked: its verdict).
__global__ __launch_bounds__(256) void index_first_round_kernel(const int32_t* __restrict__ tok, const int32_t* __restrict__ pos,
                                                                const int32_t* __restrict__ cu, int B, int N,
                                                                int32_t* __restrict__ lead, int32_t* __restrict__ first,
                                                                const int32_t* checked) {
    if (checked && checked[0] != 0) return;
    const int lane = threadIdx.x & 63;
    const int s = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (s >= B) return;
    // the first sequence that ends behind 0: one of the first 64, or searched (walked to by every wavefront, a run of empty
    // sequences in front made the launch quadratic: 999 800 of them 425 ms)
    const unsigned long long some = __ballot(cu[lane < B ? lane + 1 : B] > 0);
    const int l = some != 0ull ? __ffsll((long long)some) - 1 : first_end_behind(cu, 0, B - 1, 0, lane);
    const int bs = cu[s], es = cu[s + 1], bl = cu[l], el = cu[l + 1];
    if (s == l || bs < 0 || es <= bs || es > N || bl < 0 || el <= bl || el > N) return;
    const int len_s = es - bs, len_l = el - bl;
    const int m = common_prefix<8>(tok, pos, bs, bl, 0, len_s < len_l ? len_s : len_l, l, lead, lane);
    if (lane == 0) first[s] = m;
}

// first_done: index_first_round_kernel ran before.
// SEQ: 0, or the largest B for which the grouping table (H slots, a power of two <= 2 SEQ) and the per-sequence state live in
// LDS instead of the workspace: what one step leaves for the next is an LDS access away instead of a round trip to L2, and there are ten of those in a round.  (Two sizes: the larger one costs
// small batches 1 us.)
// 2048 sequences of 512 tokens, half of them shared: 29 us with the state in the workspace and a pass over all sequences for
// every wavefront of step 1, 15.6 with both here and a list of the followers that are left.
template <int SEQ>
__global__ __launch_bounds__(IDX_THREADS) void index_chain_kernel(
    const int32_t* __restrict__ tok, const int32_t* __restrict__ pos, const int32_t* __restrict__ cu,
    int B, int N, int32_t* __restrict__ lead, int32_t* hdr, int32_t* ldr_ws, int32_t* dep_ws, int32_t* bdep_ws,
    int32_t* mis_ws, int32_t* myslot_ws, int32_t* cbase, int32_t* slot_owner_ws, int32_t* slot_min_ws, int H,
    int32_t* n_compact_dev, int first_done, int32_t* host) {
    constexpr bool LDS = SEQ > 0;
    constexpr int LDS_TABLE = 2 * SEQ, LDS_SEQ = SEQ;
    constexpr int BATCH = LDS && SEQ <= IDX_THREADS ? 1 : 4;           // sequences that a thread fetches the state of at a time
    typedef typename std::conditional<LDS, uint16_t, int32_t>::type Index;
    __shared__ int sh_wave_tot[IDX_WAVES];
    __shared__ int sh_left[2];
    __shared__ int32_t sh_table[LDS ? 2 * LDS_TABLE : 1];
    __shared__ int32_t sh_state[LDS ? 5 * LDS_SEQ : 1];
    __shared__ uint16_t sh_list[LDS ? LDS_SEQ : 1];
    int32_t* const slot_owner = LDS ? sh_table : slot_owner_ws;
    int32_t* const slot_min = LDS ? sh_table + LDS_TABLE : slot_min_ws;
    int32_t* const ldr = LDS ? sh_state : ldr_ws;
    int32_t* const dep = LDS ? sh_state + LDS_SEQ : dep_ws;
    int32_t* const bdep = LDS ? sh_state + 2 * LDS_SEQ : bdep_ws;
    int32_t* const mis = LDS ? sh_state + 3 * LDS_SEQ : mis_ws;
    int32_t* const myslot = LDS ? sh_state + 4 * LDS_SEQ : myslot_ws;
    Index* const list = LDS ? (Index*)sh_list : (Index*)cbase;         // the followers left; cbase is not needed before the end
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < 2) sh_left[tid] = 0;
    const int s0 = index_init<BATCH>(cu, B, N, hdr, ldr, dep, bdep, mis, first_done ? mis_ws : nullptr, n_compact_dev);
    if (s0 < 0) {
        if (tid == 0) tell_host(host, RADIX_ERR_BAD_CU_SEQLENS, 0);
        return;
    }
    for (int h = tid; h < H; h += IDX_THREADS) {
        slot_owner[h] = -1;
        slot_min[h] = 0x7FFFFFFF;
    }
    __syncthreads();

    // ---- rounds.  Each active follower's matched depth grows by >= 1 per round, so the loop
    // ends after at most (longest sequence + 1) rounds; N + 2 is a hard upper bound.
    for (int round = 0; round < N + 2; ++round) {
        for (int base = 0; base < B; base += IDX_THREADS) {
            const int s = base + tid;
            const unsigned long long mine = __ballot(s < B && bdep[s < B ? s : 0] == -1);
            int at = 0;
            if (lane == 0 && mine != 0ull) at = atomicAdd(&sh_left[round & 1], __popcll(mine));
            at = __shfl(at, 0, 64) + __popcll(mine & ((1ull << lane) - 1));
            if (mine >> lane & 1) list[at] = (Index)s;
        }
        __syncthreads();
        const int left = sh_left[round & 1];
        if (left == 0) break;
        if (tid == 0) sh_left[(round + 1) & 1] = 0;

        // step 1: longest common prefix with the leader, one wavefront per follower
        if (round > 0 || !first_done) {
            for (int i = wave; i < left; i += IDX_WAVES) {
                const int s = list[i];
                const int l = ldr[s], st = dep[s];
                const int bs = cu[s], bl = cu[l];
                const int len_s = cu[s + 1] - bs, len_l = cu[l + 1] - bl;
                const int m = common_prefix<LCP_UNROLL>(tok, pos, bs, bl, st, len_s < len_l ? len_s : len_l, l, lead, lane);
                if (lane == 0) {
                    if (m == len_s) {       // s ran out while still equal to its leader: no new node
                        bdep[s] = len_s;
                        ldr[s] = -1;
                    } else {
                        mis[s] = m;         // s leaves its leader at depth m
                    }
                }
            }
            __syncthreads();
        }

        // step 2: group the leavers by (leader, depth, token, position) - exact comparison, of full keys only where the
        // 32-bit hashes agree.  dep[] holds the hash meanwhile: the depth it keeps was used in step 1 and step 3 sets
        // the next one.
        for (int i0 = tid; i0 < left; i0 += BATCH * IDX_THREADS) {
            int sq[BATCH], at[BATCH], t[BATCH], pp[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int i = i0 + u * IDX_THREADS;
                sq[u] = i < left ? (int)list[i] : -1;
                if (sq[u] >= 0 && bdep[sq[u]] != -1) sq[u] = -1;
                at[u] = sq[u] >= 0 ? cu[sq[u]] : 0;
            }
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int m = sq[u] >= 0 ? mis[sq[u]] : 0;
                t[u] = sq[u] >= 0 ? tok[at[u] + m] : 0;
                pp[u] = sq[u] >= 0 && pos ? pos[at[u] + m] : m;
            }
#pragma unroll
            for (int u = 0; u < BATCH; ++u)
                if (sq[u] >= 0) dep[sq[u]] = (int)key_hash(ldr[sq[u]], mis[sq[u]], t[u], pp[u]);
        }
        __syncthreads();
        for (int i = tid; i < left; i += IDX_THREADS) {
            const int s = list[i];
            if (bdep[s] != -1) continue;
            const int hash = dep[s];
            uint32_t h = (uint32_t)hash & (uint32_t)(H - 1);
            for (int probe = 0; probe < H; ++probe) {
                int o = LDS ? __hip_atomic_load(&slot_owner[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)
                            : ld_agent(&slot_owner[h]);
                if (o == -1) {
                    o = atomicCAS(&slot_owner[h], -1, s);
                    if (o == -1) o = s;
                }
                if (o == s) break;
                if (dep[o] == hash) {
                    const int l = ldr[s], m = mis[s], at = cu[s] + m, ot = cu[o] + m;
                    if (ldr[o] == l && mis[o] == m && tok[ot] == tok[at] && (pos == nullptr || pos[ot] == pos[at])) break;
                }
                h = (h + 1) & (uint32_t)(H - 1);
            }
            atomicMin(&slot_min[h], s);
            myslot[s] = (int)h;
        }
        __syncthreads();

        // step 3: lowest member leads the new node, the others follow it
        for (int i = tid; i < left; i += IDX_THREADS) {
            const int s = list[i];
            if (bdep[s] != -1) continue;
            const int c = LDS ? slot_min[myslot[s]] : ld_agent(&slot_min[myslot[s]]);
            const int m = mis[s];
            if (c == s) {
                bdep[s] = m;
                ldr[s] = -1;
            } else {
                ldr[s] = c;
                dep[s] = m;
            }
        }
        __syncthreads();
        for (int i = tid; i < left; i += IDX_THREADS) {
            const int s = list[i];
            if (mis[s] < 0) continue;
            const int h = myslot[s];
            slot_owner[h] = -1;
            slot_min[h] = 0x7FFFFFFF;
            mis[s] = -1;
        }
        __syncthreads();
    }

    // ---- compact-id base of every sequence: exclusive scan of its count of new nodes
    int running = 0;
    for (int base = 0; base < B; base += IDX_THREADS) {
        const int s = base + tid;
        int cnt = 0;
        if (s < B) {
            int b = bdep[s];
            int len = cu[s + 1] - cu[s];
            if (b < 0) {            // cannot happen (loop bound); keep the maps well-formed anyway
                b = len;
                bdep[s] = len;
                set_status(hdr, RADIX_ERR_BAD_SIZE);
                sh_left[0] = RADIX_ERR_BAD_SIZE;
            }
            if (LDS) bdep_ws[s] = b;
            cnt = len - b;
        }
        int incl = cnt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            int v = __shfl_up(incl, o, 64);
            if (lane >= o) incl += v;
        }
        if (lane == 63) sh_wave_tot[wave] = incl;
        __syncthreads();
        int before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < IDX_WAVES; ++w) {
            int v = sh_wave_tot[w];
            if (w < wave) before += v;
            total += v;
        }
        if (s < B) cbase[s] = running + before + incl - cnt;
        running += total;
        __syncthreads();
    }
    if (tid == 0) {
        *n_compact_dev = running;
        hdr[1] = running;
        hdr[2] = s0;
        tell_host(host, sh_left[0] < 0 ? sh_left[0] : 0, running);
    }
}

// U original positions per thread, 64 U consecutive ones per wavefront: turn (leader sequence, offset) into compact ids.  What
// bounds it is memory latency: the sequence of a position used to be searched by every thread on its own, eleven dependent loads
// for 2048 sequences.  Now the wavefront searches the sequence of its first position, 64 candidates a step, and the few ends of
// sequences behind it come with one more load; only where 64 sequences or more end within them every lane searches for
// itself.  1 050 931 tokens in 2048 sequences: 12.7 -> 7.0 us.
template <int U>
__global__ __launch_bounds__(256) void index_finalize_kernel(
    const int32_t* __restrict__ tok, const int32_t* __restrict__ pos, const int32_t* __restrict__ cu,
    int B, int N, int32_t* __restrict__ I_scatter /* holds leader ids of duplicate positions, those below first[s] apart */,
    int32_t* __restrict__ I_gather, int32_t* hdr, const int32_t* __restrict__ bdep,
    const int32_t* __restrict__ cbase, const int32_t* __restrict__ first, int32_t* host) {
    if (ld_agent(&hdr[0]) == RADIX_ERR_BAD_CU_SEQLENS) return;
    const int lane = threadIdx.x & 63;
    const int j0 = blockIdx.x * (256 * U) + (threadIdx.x >> 6) * (64 * U);
    if (j0 >= N) return;
    const int left = N - j0, j_last = left > 64 * U ? j0 + 64 * U - 1 : N - 1;
    int t[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = 64 * u + lane;
        t[u] = i < left ? tok[j0 + i] : 0;
        if (pos != nullptr && i < left) t[u] |= pos[j0 + i];     // negative if one of the two is
    }
    const int s0 = first_end_behind(cu, 0, B - 1, j0, lane);       // it exists, as cu[B] = N
    const int i_end = s0 + 1 + lane;
    const int end = i_end <= B ? cu[i_end] : 0x7FFFFFFF;    // ends of the sequences s0, s0 + 1, ...
    const unsigned long long inside = __ballot(end <= j_last);
    const int n_in = __popcll(inside);
    int sq[U];
    if (n_in < 64) {
#pragma unroll
        for (int u = 0; u < U; ++u) sq[u] = s0;
        for (int k = 0; k < n_in; ++k) {
            const int e = __shfl(end, k, 64);
#pragma unroll
            for (int u = 0; u < U; ++u) sq[u] += e - j0 <= 64 * u + lane;
        }
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = 64 * u + lane < left ? j0 + 64 * u + lane : N - 1;
            int a = s0, b = B - 1;
            while (a < b) {
                const int mid = (a + b) >> 1;
                if (cu[mid + 1] > j) b = mid; else a = mid + 1;
            }
            sq[u] = a;
        }
    }
    int p[U], bd[U], cb[U], ld[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = 64 * u + lane, s = sq[u];
        p[u] = j0 - cu[s] + i;
        bd[u] = bdep[s];
        cb[u] = cbase[s];
        ld[u] = -1;
        if (i < left && p[u] < bd[u]) ld[u] = first && p[u] < first[s] ? hdr[2] : I_scatter[j0 + i];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (64 * u + lane >= left) continue;
        const int j = j0 + 64 * u + lane;
        if (t[u] < 0 && atomicCAS(hdr, 0, RADIX_ERR_BAD_TOKEN) == 0 && host)
            __hip_atomic_store(host, RADIX_ERR_BAD_TOKEN, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        if (ld[u] < 0) {
            const int c = cb[u] + (p[u] - bd[u]);
            I_scatter[j] = c;
            I_gather[c] = j;
        } else {
            I_scatter[j] = cbase[ld[u]] + (p[u] - bdep[ld[u]]);
        }
    }
}

int next_pow2(int x) {
    int h = 64;
    while (h < x) h <<= 1;
    return h;
}

}  // namespace

size_t radix_index_ws_bytes(int B) {
    size_t H = (size_t)next_pow2(2 * (B > 0 ? B : 1));
    return RADIX_WS_HEADER_BYTES + align_up(((size_t)6 * (size_t)(B > 0 ? B : 1) + 2 * H) * sizeof(int32_t), 256);
}

extern "C" int radix_index_workspace_bytes(int32_t max_B, size_t* bytes_out) {
    if (!bytes_out) return RADIX_ERR_NULL_POINTER;
    if (max_B < 0) return RADIX_ERR_BAD_SIZE;
    *bytes_out = radix_index_ws_bytes(max_B);
    return RADIX_OK;
}

namespace {

// Whether the comparisons of the first round get a launch over the whole chip (one launch more, 2 us).  In the chain
// kernel IDX_WAVES followers are compared at a time; every further step of that loop costs 0.9 us and 4 ns per token
// compared.  How many tokens that will be is not known before; half of the mean length is counted.  The line lies above
// break-even, which keeps batches that share less from losing.  Measured (us, one kernel / over the chip): 24 sequences of a
// shared prefix of 16 tokens 30.4 / 32.7, of 512 tokens 34.6 / 33.9, of 2048 tokens 45.5 / 39.1; 48 of 16 tokens 33.0 / 34.2, of
// 1024 43.9 / 35.7; 64 of 16 tokens 34.9 / 35.7, of 512 43.3 / 36.4; 96 of 16 tokens 36.0 / 34.8; nothing shared, 48 of 450
// tokens 32.2 / 32.7.
bool first_round_over_the_chip(int B, int N) {
    if (B <= IDX_WAVES) return false;
    const long long more_steps = (B - 2) / IDX_WAVES;           // B - 1 followers
    return more_steps * (900 + 4 * (long long)(N / B) / 2) >= 4500;
}

// Words of pinned host memory that the kernels write a call's status and N' to, so that the host that waits for them needs no copy
// behind the kernels (2048 x 512 tokens 56 -> 47 us a call, 8 x 48 about 8 us less).  One page for the process, made on the first such
// call and kept; a call borrows
// one of its 64 slots, and copies as before if there is none.
struct HostSlots {
    static constexpr int SLOT_WORDS = 16;                       // one cache line each
    std::mutex m;
    int32_t* page = nullptr;
    bool made = false;
    uint64_t taken = 0;
    int borrow(int32_t** words) {
        std::lock_guard<std::mutex> lock(m);
        if (!made) {
            made = true;
            // the allocation must not end a capture that some other thread has under way
            hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
            if (hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess) {
                if (hipHostMalloc((void**)&page, 64 * SLOT_WORDS * sizeof(int32_t), hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) {
                    page = nullptr;
                    (void)hipGetLastError();
                }
                (void)hipThreadExchangeStreamCaptureMode(&mode);
            }
        }
        if (!page || taken == ~0ull) return -1;
        const int i = __builtin_ctzll(~taken);
        taken |= 1ull << i;
        *words = page + i * SLOT_WORDS;
        return i;
    }
    void give_back(int i) {
        std::lock_guard<std::mutex> lock(m);
        taken &= ~(1ull << i);
    }
    int available() {
        std::lock_guard<std::mutex> lock(m);
        return page ? 64 - __builtin_popcountll(taken) : 0;
    }
};
HostSlots& host_slots() {
    static HostSlots* const s = new HostSlots;                  // never destroyed: the runtime may be gone before static objects are
    return *s;
}

// A call inside a capture cannot wait (it fails where it tries to): no slot for it, or that one could never be given back.
bool waiting_is_possible(hipStream_t stream) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) == hipSuccess) return status == hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return false;
}

// may_allocate: false for the entry point that promises not to
int build_index_impl(const int32_t* tok, const int32_t* pos, const int32_t* cu_seqlens, int32_t B, int32_t N,
                     int32_t* I_scatter, int32_t* I_gather, int32_t* n_compact_dev, int32_t* n_compact_host,
                     void* ws, hipStream_t stream, bool may_allocate) {
    int32_t* hdr = (int32_t*)ws;
    int32_t* base = (int32_t*)((char*)ws + RADIX_WS_HEADER_BYTES);
    const size_t Bn = (size_t)(B > 0 ? B : 1);
    const int H = next_pow2(2 * (int)Bn);
    int32_t* ldr = base;
    int32_t* dep = ldr + Bn;
    int32_t* bdep = dep + Bn;
    int32_t* mis = bdep + Bn;
    int32_t* myslot = mis + Bn;
    int32_t* cbase = myslot + Bn;
    int32_t* slot_owner = cbase + Bn;
    int32_t* slot_min = slot_owner + H;

    // The launches of one call together initialise every word of builder state that they read, so the buffer may hold
    // anything when the call starts: index_first_round_kernel writes where the followers leave, the chain kernel the status word,
    // the per-sequence state and its slot table (in LDS up to LDS_SEQ_MANY sequences; the arrays in the workspace are for larger
    // batches).
    const int first_done = N > 0 && first_round_over_the_chip(B, N);
    int32_t* host = nullptr;
    const int slot = n_compact_host && may_allocate && waiting_is_possible(stream) ? host_slots().borrow(&host) : -1;
    const bool in_lds = B <= LDS_SEQ_MANY;              // then the chain kernel leaves mis[] as the first round wrote it
    if (first_done) {
        if (!in_lds) hipLaunchKernelGGL(index_check_kernel, dim3(1), dim3(IDX_THREADS), 0, stream, cu_seqlens, B, N, hdr);
        hipLaunchKernelGGL(index_first_round_kernel, dim3(ceil_div(B, 4)), dim3(256), 0, stream, tok, pos, cu_seqlens, B, N,
                           in_lds ? nullptr : I_scatter, mis, in_lds ? nullptr : hdr);
    }
    auto chain = B <= LDS_SEQ_FEW ? index_chain_kernel<LDS_SEQ_FEW> : B <= LDS_SEQ_MANY ? index_chain_kernel<LDS_SEQ_MANY> : index_chain_kernel<0>;
    hipLaunchKernelGGL(chain, dim3(1), dim3(IDX_THREADS), 0, stream, tok, pos, cu_seqlens, B, N, I_scatter,
                       hdr, ldr, dep, bdep, mis, myslot, cbase, slot_owner, slot_min, H, n_compact_dev, first_done, host);
    if (N > 0) {
        // few: workgroups for every CU come first; nor may the count of workgroups leave 32 bits
        const bool few = N < 1 << 18 || N > 0x7FFFFFFF - 1023;
        auto finalize = few ? index_finalize_kernel<1> : index_finalize_kernel<4>;
        hipLaunchKernelGGL(finalize, dim3(ceil_div(N, few ? 256 : 1024)), dim3(256), 0, stream, tok, pos,
                           cu_seqlens, B, N, I_scatter, I_gather, hdr, bdep, cbase, first_done && in_lds ? mis : nullptr, host);
    }
    const hipError_t launched = hipGetLastError();
    if (n_compact_host) {
        int32_t h2[2] = {0, 0};
        if (slot >= 0) {
            // whatever went wrong, the words go back only when nothing on the stream can write them any more
            const hipError_t waited = hipStreamSynchronize(stream);
            if (launched == hipSuccess && waited == hipSuccess) {
                h2[0] = __atomic_load_n(host, __ATOMIC_ACQUIRE);
                h2[1] = __atomic_load_n(host + 1, __ATOMIC_ACQUIRE);
            }
            if (waited == hipSuccess) host_slots().give_back(slot);
            if (launched != hipSuccess || waited != hipSuccess) return RADIX_ERR_HIP;
        } else {
            if (launched != hipSuccess) return RADIX_ERR_HIP;
            HIP_TRY(hipMemcpyAsync(h2, hdr, sizeof(h2), hipMemcpyDeviceToHost, stream));
            HIP_TRY(hipStreamSynchronize(stream));
        }
        *n_compact_host = h2[1];
        if (h2[0] != 0) return h2[0];
        return RADIX_OK;
    }
    return launched == hipSuccess ? RADIX_OK : RADIX_ERR_HIP;
}

int check_index_args(const int32_t* tok, const int32_t* cu_seqlens, int32_t B, int32_t N, const int32_t* I_scatter,
                     const int32_t* I_gather, const int32_t* n_compact_dev) {
    if (B < 0 || N < 0) return RADIX_ERR_BAD_SIZE;
    if (B > (1 << 28)) return RADIX_ERR_BAD_SIZE;
    if (!cu_seqlens || !n_compact_dev) return RADIX_ERR_NULL_POINTER;
    if (N > 0 && (!tok || !I_scatter || !I_gather)) return RADIX_ERR_NULL_POINTER;
    if (N > 0 && B == 0) return RADIX_ERR_BAD_SIZE;
    return RADIX_OK;
}

}  // namespace

extern "C" int radix_debug_index_first_round(int32_t B, int32_t N) {
    if (B <= 0 || N <= 0) return RADIX_ERR_BAD_SIZE;
    return first_round_over_the_chip(B, N) ? 1 : 0;
}

extern "C" int radix_debug_index_host_slots(void) { return host_slots().available(); }

extern "C" int radix_build_index(const int32_t* tok, const int32_t* pos, const int32_t* cu_seqlens,
                                 int32_t B, int32_t N, int32_t* I_scatter, int32_t* I_gather,
                                 int32_t* n_compact_dev, int32_t* n_compact_host,
                                 void* ws, size_t ws_bytes, void* stream) {
    const int rc = check_index_args(tok, cu_seqlens, B, N, I_scatter, I_gather, n_compact_dev);
    if (rc != RADIX_OK) return rc;
    if (!ws) return RADIX_ERR_NULL_POINTER;
    if (((uintptr_t)ws & 255) != 0) return RADIX_ERR_MISALIGNED;
    if (ws_bytes < radix_index_ws_bytes(B)) return RADIX_ERR_WORKSPACE_TOO_SMALL;
    return build_index_impl(tok, pos, cu_seqlens, B, N, I_scatter, I_gather, n_compact_dev, n_compact_host, ws,
                            (hipStream_t)stream, true);
}

// ---- the same builder for callers that cannot allocate: its state lives in a static device array
// instead of a caller-provided workspace.  Every GPU the library runs on holds its own copy of the
// array at its own address; host code only ever uses the address hipGetSymbolAddress reports for
// the current device (the array's name is not a device address on the host side).
namespace {

constexpr size_t STATIC_INDEX_BYTES =
    RADIX_WS_HEADER_BYTES + ((size_t)6 * RADIX_STATIC_INDEX_MAX_B + 2 * (size_t)(2 * RADIX_STATIC_INDEX_MAX_B)) * sizeof(int32_t);
static_assert((RADIX_STATIC_INDEX_MAX_B & (RADIX_STATIC_INDEX_MAX_B - 1)) == 0 && RADIX_STATIC_INDEX_MAX_B >= 64,
              "the slot tables hold next_pow2(2 B) entries each");
static __device__ __align__(256) unsigned char scratch[STATIC_INDEX_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[MAX_DEVICES] = {};

// address of `scratch` on the current device, looked up once per device
int static_scratch(void** out) {
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return RADIX_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return RADIX_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return RADIX_OK;
}

}  // namespace

extern "C" int radix_build_index_static(const int32_t* tok, const int32_t* pos, const int32_t* cu_seqlens,
                                        int32_t B, int32_t N, int32_t* I_scatter, int32_t* I_gather,
                                        int32_t* n_compact_dev, int32_t* n_compact_host, void* stream) {
    int rc = check_index_args(tok, cu_seqlens, B, N, I_scatter, I_gather, n_compact_dev);
    if (rc != RADIX_OK) return rc;
    if (B > RADIX_STATIC_INDEX_MAX_B) return RADIX_ERR_STATIC_LIMIT;
    void* ws = nullptr;
    if ((rc = static_scratch(&ws)) != RADIX_OK) return rc;
    return build_index_impl(tok, pos, cu_seqlens, B, N, I_scatter, I_gather, n_compact_dev, n_compact_host, ws,
                            (hipStream_t)stream, false);
}
