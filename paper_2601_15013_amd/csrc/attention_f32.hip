// fp32 causal varlen GQA attention for the fp32 model configuration (small, parity-oriented).
// One wavefront per (query token, query head): keys are visited 64 at a time with an online
// softmax; lane e accumulates output elements e and e + 64 (head_dim <= 128).
// (Paper: Algorithm 1, "FlashAttn(q, k, v, cu_seqlens, causal=True)" on the full layout.)
// With maps, scatter and gather are folded in: q, k and v rows are read from the compact buffer through I_scatter and only the
// representative tokens are computed; a row's arithmetic is the same, so its values are, too.
//
// What bounds it is latency: a row is one wavefront that walks its keys alone.  So the 16 key pieces of a lane and the value rows,
// 16 at a time and 16 ahead, are in flight together.  Batch of 8 sequences of 32 shared + 16 own tokens, 4 heads of 64: 10.1 us on
// the full layout with 8 rows at a time, 8.2 us like this, and the two row copies around it (2.7 us each) are gone.  64 sequences of
// 256 shared + 64 own tokens: the forward 1449 -> 730 us.
#include "common.h"
#include "kernels.h"

namespace {

template <bool WIDE>                                // head_dim > 64
__global__ __launch_bounds__(64) void attention_f32_kernel(const float* __restrict__ qkv, const int32_t* __restrict__ cu,
                                                           int B, int N, int n_q_heads, int n_kv_heads, int hd,
                                                           float* __restrict__ out, AttnF32Maps maps) {
    constexpr int VB = 16;                          // value rows per batch
    __shared__ __attribute__((aligned(16))) float qs[128];
    __shared__ float ps[64];
    const int lane = threadIdx.x;
    const int h = blockIdx.y;          // query head
    const int g = h / (n_q_heads / n_kv_heads);
    const int dq = n_q_heads * hd, dkv = n_kv_heads * hd;
    const int row = dq + 2 * dkv;
    int i = blockIdx.x;                // query token (original layout)
    if (maps.gather) {
        i = (int)blockIdx.x < maps.n_compact ? maps.gather[blockIdx.x] : 0;
        if (i < 0 || i >= N) {
            if (lane == 0) set_status(maps.status, RADIX_ERR_BAD_TOKEN);
            i = i < 0 ? 0 : N - 1;
        }
    }
    auto source = [&](int j) {         // row of qkv that holds token j
        if (!maps.gather) return j;
        int c = maps.scatter[j];
        if (c < 0 || c >= maps.n_compact) {
            set_status(maps.status, RADIX_ERR_BAD_TOKEN);
            c = c < 0 ? 0 : maps.n_compact - 1;
        }
        return c;
    };
    int lo = 0, hi = B - 1;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (cu[mid + 1] > i) hi = mid; else lo = mid + 1;
    }
    int start = cu[lo];
    start = start < 0 ? 0 : (start > i ? i : start);    // a malformed cu_seqlens cannot leave the N rows
    const float scale = 1.0f / sqrtf((float)hd);
    const size_t qrow = (size_t)source(i);
    for (int e = lane; e < hd; e += 64) qs[e] = qkv[qrow * row + h * hd + e] * scale;
    __syncthreads();
    // output elements of this lane; lanes past the head repeat its last one and store nothing
    const int e0 = lane < hd ? lane : hd - 1, e1 = lane + 64 < hd ? lane + 64 : hd - 1;
    float m = -INFINITY, l = 0.f, acc0 = 0.f, acc1 = 0.f;
    for (int j0 = start; j0 <= i; j0 += 64) {
        const int j = j0 + lane;
        const int cnt = (i - j0 + 1) < 64 ? (i - j0 + 1) : 64;
        const int src = source(j <= i ? j : i);
        const float* vb = qkv + dq + dkv + g * hd;
        // value rows t0 .. t0 + VB - 1 of the chunk (past its end: the last one again)
        float v0[2][VB], v1[2][VB];
        auto fetch_v = [&](int t0, float (&a)[VB], float (&b)[VB]) {
#pragma unroll
            for (int u = 0; u < VB; ++u) {
                const int t = t0 + u < cnt ? t0 + u : cnt - 1;
                const float* vr = vb + (size_t)__builtin_amdgcn_readlane(src, t) * row;
                a[u] = vr[e0];
                if (WIDE) b[u] = vr[e1];
            }
        };
        float s = -INFINITY;
        {
            const float* kr = qkv + (size_t)src * row + dq + g * hd;      // 16-byte aligned: hd is a multiple of 4
            float dot = 0.f;
#pragma unroll 16
            for (int e = 0; e < hd; e += 4) {
                const f32x4 k4 = *reinterpret_cast<const f32x4*>(kr + e);
                const f32x4 q4 = *reinterpret_cast<const f32x4*>(qs + e);
#pragma unroll
                for (int u = 0; u < 4; ++u) dot = fmaf(q4[u], k4[u], dot);
            }
            if (j <= i) s = dot;
        }
        fetch_v(0, v0[0], v1[0]);
        const float m_new = fmaxf(m, wave_max(s));
        const float p = (j <= i) ? expf(s - m_new) : 0.f;
        const float alpha = expf(m - m_new);        // m = -inf on the first chunk: alpha = 0
        l = l * alpha + wave_sum(p);
        acc0 *= alpha; acc1 *= alpha;
        m = m_new;
        __syncthreads();
        ps[lane] = p;
        __syncthreads();
#pragma unroll
        for (int b = 0; b < 64 / VB; ++b) {
            if (b * VB >= cnt) break;
            if ((b + 1) * VB < cnt) fetch_v((b + 1) * VB, v0[(b + 1) & 1], v1[(b + 1) & 1]);
#pragma unroll
            for (int u = 0; u < VB; ++u) {
                if (b * VB + u >= cnt) break;
                acc0 = fmaf(ps[b * VB + u], v0[b & 1][u], acc0);
                if (WIDE) acc1 = fmaf(ps[b * VB + u], v1[b & 1][u], acc1);
            }
        }
    }
    float* o = out + (size_t)blockIdx.x * dq + h * hd;
    if (lane < hd) o[lane] = acc0 / l;
    if (WIDE && lane + 64 < hd) o[lane + 64] = acc1 / l;
}

}  // namespace

void launch_attention_f32(const float* qkv, const int32_t* cu, int B, int N, int n_rows, int n_q_heads, int n_kv_heads, int hd,
                          float* out, const AttnF32Maps& maps, hipStream_t stream) {
    if (N <= 0 || n_rows <= 0) return;
    auto kernel = hd > 64 ? attention_f32_kernel<true> : attention_f32_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3(n_rows, n_q_heads), dim3(64), 0, stream, qkv, cu, B, N, n_q_heads, n_kv_heads, hd, out, maps);
}
