// fp32 GEMM C[M, Nout] = A[M, K] * W[Nout, K]^T for the fp32 model configuration (small,
// parity-oriented).  LDS-tiled FMA kernel, K consumed in order by one fused multiply-add chain per output element,
// so every element is reduced in the same order whatever the tile and wherever its row sits in the matrix.
//
// Two regimes.  With few rows the launch is latency-bound: a few dozen workgroups, and the time is the number of k-tiles
// times what one costs.  So the outputs of a tile are TM x TM with TM = 16 R, the smaller the fewer workgroups there
// are, the k-tile of the small ones is 64 wide, the next one is fetched into registers (16 bytes per lane) while the
// present one is multiplied, and LDS is read 16 bytes along k.  M 300, K 768, N 256: 27.9 us with R = 2, against 88.5 us
// with a 64 x 64 tile of scalar LDS reads, k-tiles of 16 and no prefetch.  SwiGLU needs gate and up columns in one tile: the
// smallest one is 16 rows of 16 + 16 columns (M 160, N 1536, K 256: 14.1 us with 32 x 32, 7.4 with it).
// With many rows every CU has several workgroups that hide each other's latency, and what counts is how many fit: the
// 64 x 64 tile (R = 4) takes k-tiles of 16 (10 KB of LDS and 88 registers against 35 KB and 116 with k-tiles of 64).
// us with k-tiles of 64 / 32 / 16 / the kernel of scalar reads: M 24000 N 1536 K 256 (gate/up) 410 / 377 / 270 / 345;
// M 65000 N 256 K 768 641 / 595 / 355 / 478 (72 TFLOP/s); M 12000 N 6144 K 1024 3066 / 2912 / 1902 / 2444 (79 TFLOP/s).
#include "common.h"
#include "kernels.h"

namespace {

// 256 threads = 16 x 16; thread (tx, ty) owns rows ty + 16 i, i < RM, and columns tx + 16 j, j < R.
template <int RM, int R, int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ W,
                                                       int M, int Nout, int K, float* __restrict__ out) {
    static_assert(EPI != EPI_SWIGLU || R == 4 || R == 2, "gate and up blocks of 32 columns meet in one tile");
    // SwiGLU with a 32-wide tile takes 16 gate columns and the 16 matching up columns, else 64 = 32 gate + 32 up
    constexpr bool PAIR16 = EPI == EPI_SWIGLU && R == 2;
    constexpr int TK = RM == 4 ? 16 : 64, PK = TK + 4;      // k-tile and its pitch in LDS: 16 rows start in 16 different 16-byte bank groups
    constexpr int TM = 16 * RM, TN = 16 * R, LA = TM * TK / 4 / 256, LW = TN * TK / 4 / 256;
    static_assert(LA >= 1 && LA * 256 * 4 == TM * TK && LW * 256 * 4 == TN * TK, "every thread fetches whole pieces of 16 bytes");
    __shared__ float As[TM * PK];
    __shared__ float Ws[TN * PK];
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    const int m0 = blockIdx.y * TM;
    // weight row of tile column c
    const int n0 = PAIR16 ? ((int)blockIdx.x >> 1) * 64 + ((int)blockIdx.x & 1) * 16 : (int)blockIdx.x * TN;
    auto w_row = [&](int c) { return PAIR16 ? n0 + (c & 15) + (c >> 4) * 32 : n0 + c; };
    float4 av[LA], wv[LW];
    auto piece = [](const float* p, bool inside) {
        // by value: `inside ? *p : zero` with a named zero selects between two addresses, which puts zero into scratch memory and
        // makes the load a flat one
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (inside) v = *reinterpret_cast<const float4*>(p);
        return v;
    };
    auto fetch = [&](int k0) {                                   // K is a multiple of 4, rows are 16-byte aligned
#pragma unroll
        for (int u = 0; u < LA; ++u) {
            const int e = tid + 256 * u, gm = m0 + e / (TK / 4), gk = k0 + 4 * (e % (TK / 4));
            av[u] = piece(A + (size_t)gm * K + gk, gm < M && gk < K);
        }
#pragma unroll
        for (int u = 0; u < LW; ++u) {
            const int e = tid + 256 * u, gn = w_row(e / (TK / 4)), gk = k0 + 4 * (e % (TK / 4));
            wv[u] = piece(W + (size_t)gn * K + gk, gn < Nout && gk < K);
        }
    };
    float acc[RM][R] = {};
    fetch(0);
    for (int k0 = 0; k0 < K; k0 += TK) {
#pragma unroll
        for (int u = 0; u < LA; ++u) {
            const int e = tid + 256 * u;
            *reinterpret_cast<float4*>(As + e / (TK / 4) * PK + 4 * (e % (TK / 4))) = av[u];
        }
#pragma unroll
        for (int u = 0; u < LW; ++u) {
            const int e = tid + 256 * u;
            *reinterpret_cast<float4*>(Ws + e / (TK / 4) * PK + 4 * (e % (TK / 4))) = wv[u];
        }
        __syncthreads();
        if (k0 + TK < K) fetch(k0 + TK);
#pragma unroll
        for (int k = 0; k < TK; k += 4) {
            float4 a[RM], b[R];
#pragma unroll
            for (int i = 0; i < RM; ++i) a[i] = *reinterpret_cast<const float4*>(As + (ty + 16 * i) * PK + k);
#pragma unroll
            for (int j = 0; j < R; ++j) b[j] = *reinterpret_cast<const float4*>(Ws + (tx + 16 * j) * PK + k);
#pragma unroll
            for (int i = 0; i < RM; ++i)
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    acc[i][j] = fmaf(a[i].x, b[j].x, acc[i][j]);
                    acc[i][j] = fmaf(a[i].y, b[j].y, acc[i][j]);
                    acc[i][j] = fmaf(a[i].z, b[j].z, acc[i][j]);
                    acc[i][j] = fmaf(a[i].w, b[j].w, acc[i][j]);
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < RM; ++i) {
        const int gm = m0 + ty + 16 * i;
        if (gm >= M) continue;
        if (EPI == EPI_SWIGLU) {
            // tile columns [0, TN / 2) are gate, the others the matching up columns
#pragma unroll
            for (int j = 0; j < R / 2; ++j) {
                const int gn = w_row(tx + 16 * j);              // gate row of W; its up row is gn + 32
                if (gn + 32 < Nout) {
                    const float gte = acc[i][j], up = acc[i][j + R / 2];
                    out[(size_t)gm * (Nout >> 1) + (gn >> 6) * 32 + (gn & 31)] = gte / (1.0f + expf(-gte)) * up;
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int gn = n0 + tx + 16 * j;
                if (gn >= Nout) continue;
                float* o = out + (size_t)gm * Nout + gn;
                if (EPI == EPI_RESIDUAL) *o = *o + acc[i][j]; else *o = acc[i][j];
            }
        }
    }
}

template <int RM, int R, int EPI>
void launch_r(const float* A, const float* W, int M, int Nout, int K, float* out, hipStream_t stream) {
    const int tiles_m = ceil_div(M, 16 * RM);
    // SwiGLU columns come in blocks of 64 (32 gate + 32 up)
    const int tiles_n = EPI == EPI_SWIGLU ? ceil_div(Nout, 64) * (4 / R) : ceil_div(Nout, 16 * R);
    // the grid's y extent is 16 bits: taller outputs go in several launches
    for (int t0 = 0; t0 < tiles_m; t0 += 65535) {
        const int rows0 = t0 * 16 * RM, n = tiles_m - t0 < 65535 ? tiles_m - t0 : 65535;
        hipLaunchKernelGGL((gemm_f32_kernel<RM, R, EPI>), dim3(tiles_n, n), dim3(256), 0, stream, A + (size_t)rows0 * K, W,
                           M - rows0, Nout, K, out + (size_t)rows0 * (EPI == EPI_SWIGLU ? Nout / 2 : Nout));
    }
}

// Tile by workgroup count: the largest one reads LDS least per multiply-add, the smaller ones shorten the walk along K
// while CUs would be idle.  Measured at the line between 64 x 64 and 32 x 32 tiles (us): 176 large tiles 67.4 / 62.9 (M 700, N
// 1024, K 1024) and 194 / 173 (K 3072), 192 tiles 18.7 / 19.9 (M 1500, N 512, K 256), 240 tiles 65.3 / 80.2 (M 300, N 3072,
// K 1024).
template <int EPI>
void launch_epi(const float* A, const float* W, int M, int Nout, int K, float* out, hipStream_t stream) {
    const long long t64 = (long long)ceil_div(M, 64) * ceil_div(Nout, 64), t32 = (long long)ceil_div(M, 32) * ceil_div(Nout, 32);
    if (t64 >= 192) launch_r<4, 4, EPI>(A, W, M, Nout, K, out, stream);
    else if (t32 >= 256) launch_r<2, 2, EPI>(A, W, M, Nout, K, out, stream);
    else launch_r<1, EPI == EPI_SWIGLU ? 2 : 1, EPI>(A, W, M, Nout, K, out, stream);      // SwiGLU: gate and up columns in one tile
}

}  // namespace

void launch_gemm_f32(const float* A, const float* W, int M, int Nout, int K, int epilogue, float* out,
                     hipStream_t stream) {
    if (M <= 0 || Nout <= 0) return;
    if (epilogue == EPI_STORE) launch_epi<EPI_STORE>(A, W, M, Nout, K, out, stream);
    else if (epilogue == EPI_RESIDUAL) launch_epi<EPI_RESIDUAL>(A, W, M, Nout, K, out, stream);
    else launch_epi<EPI_SWIGLU>(A, W, M, Nout, K, out, stream);
}
