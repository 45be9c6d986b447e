// fp64 GEMM on the CDNA matrix cores (v_mfma_f64_16x16x4_f64) for the general-block form of the shared-Hinv
// elimination (Eq. 12 applied B columns at a time).
//
// One workgroup = 512 threads = 8 wavefronts computes a 64 x 64 tile of C; each wavefront owns a
// 16 x 32 part = 1 x 2 MFMA tiles (two wavefronts per SIMD: one alone issues an fp64 MFMA only every
// ~140 cycles, two interleave to the pipe's rate of one per ~64).  K is walked in chunks of
// 64: a chunk of both operand tiles is fetched with one round of loads (lane index
// along the contiguous dimension), held in registers while the previous chunk is
// multiplied out of LDS (32 MFMAs per wavefront, about one memory round trip), and
// then stored to LDS.  The C tile is prefetched with the first chunk.  The rank-64
// updates (K = 64) are latency bound -- a few tiles per launch -- so a single
// exposed memory round trip is what matters there.
#include "fobq_internal.h"

namespace fobq {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int GT = 512;   // threads per workgroup
constexpr int TM = 64, TN = 64, K1 = 64, K1_LD = K1 + 2;   // +2 doubles: conflict-free 8-byte fragment reads

template <bool TA>
__global__ __launch_bounds__(GT) void gemm64_kernel(GemmP p)
{
    const int M = p.M, N = p.N, K = p.K;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TN;
    if (p.upper && n0 + TN - 1 < m0) return;

    const double* __restrict__ A = p.A;
    const double* __restrict__ B = p.B;
    double* C = p.C;
    double* C2 = p.C2;

    __shared__ double As[TM][K1_LD];
    __shared__ double Bs[TN][K1_LD];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wr = wave >> 1, wn = wave & 1;     // 16-row slice, 32-column half of the tile

    double ra[8], rb[8];
    auto gload = [&](int kk) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int x = lane, y = wave + 8 * u;    // x: contiguous index, y: strided index (0..63)
            if (!TA) { const int gm = m0 + y, gk = kk + x; ra[u] = (gm < M && gk < K) ? A[(int64_t)gm * p.lda + gk] : 0.0; }
            else     { const int gm = m0 + x, gk = kk + y; ra[u] = (gm < M && gk < K) ? A[(int64_t)gk * p.lda + gm] : 0.0; }
            const int gn = n0 + x, gk = kk + y;
            rb[u] = (gn < N && gk < K) ? B[(int64_t)gk * p.ldb + gn] : 0.0;
        }
    };
    auto sstore = [&]() {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int x = lane, y = wave + 8 * u;
            if (!TA) As[y][x] = ra[u]; else As[x][y] = ra[u];
            Bs[x][y] = rb[u];
        }
    };

    gload(0);
    d4 cin[2];
    const bool use_c = p.beta != 0.0;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int gm = m0 + wr * 16 + 4 * v + (lane >> 4);
            const int gn = n0 + wn * 32 + j * 16 + (lane & 15);
            cin[j][v] = (use_c && gm < M && gn < N) ? C[(int64_t)gm * p.ldc + gn] : 0.0;
        }

    d4 acc[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[j] = d4{0.0, 0.0, 0.0, 0.0};

    for (int kk = 0; kk < K; kk += K1) {
        __syncthreads();                      // previous chunk fully consumed
        sstore();
        __syncthreads();
        if (kk + K1 < K) gload(kk + K1);   // in flight while this chunk is multiplied
        const int ksteps = (min(K1, K - kk) + 3) / 4;
        for (int ks = 0; ks < ksteps; ++ks) {
            const double a = As[wr * 16 + (lane & 15)][ks * 4 + (lane >> 4)];
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Bs[wn * 32 + j * 16 + (lane & 15)][ks * 4 + (lane >> 4)],
                                                              acc[j], 0, 0, 0);
        }
    }

    // accumulator layout of v_mfma_f64_16x16x4_f64: lane l, element v holds D[4 * v + l / 16][l % 16]
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int gm = m0 + wr * 16 + 4 * v + (lane >> 4);
            const int gn = n0 + wn * 32 + j * 16 + (lane & 15);
            if (gm < M && gn < N) {
                const int64_t off = (int64_t)gm * p.ldc + gn;
                double r = p.alpha * acc[j][v];
                if (use_c) r += p.beta * cin[j][v];
                C[off] = r;
                if (C2) C2[off] = p.rowscale[gm] * r;
            }
        }
}

hipError_t gemm64(hipStream_t s, const GemmP& p, bool TA)
{
    if (p.M <= 0 || p.N <= 0) return hipSuccess;
    dim3 grid((p.N + TN - 1) / TN, (p.M + TM - 1) / TM), block(GT);
    if (TA) hipLaunchKernelGGL(gemm64_kernel<true>, grid, block, 0, s, p);
    else hipLaunchKernelGGL(gemm64_kernel<false>, grid, block, 0, s, p);
    return hipGetLastError();
}

}  // namespace fobq
