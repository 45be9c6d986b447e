// Factorizations of the path, fp64, blocked with 64-wide panels (the damped inverse is in flow.hip):
//   eliminate_blocked the shared-Hinv elimination of Eq. 12, B columns at a time, for any B and any number of steps
//                    (flow.hip has the form for all columns at B = 64):
//                    after column t is processed, Hinv -= Hinv[:,t] Hinv[t,:] / Hinv[t,t].
//                    The pivot rows are kept:  U[t, t:]  = Hinv^(t)[t, t:]  and
//                    Un[t, :] = U[t, :] / U[t, t]; the weight compensation of Eq. 9 / 11
//                    for step t is  W[:, k] -= (w_t - q_t) * Un[t, k].
//   batch_*          the factor path of many small layers, one workgroup per layer
// The 64 x 64 diagonal blocks are handled by one workgroup in LDS (tile_block.h); everything
// else is products on the matrix cores (gemm64, tile_mm).
#include <hip/hip_ext.h>

#include "fobq_internal.h"
#include "tile_block.h"

namespace fobq {

__device__ __forceinline__ void elim_block_store(const double* Am, const double* Xm, const double* rv,
                                                 int64_t ld, int o, int nb, double* __restrict__ U,
                                                 double* __restrict__ Un, double* __restrict__ G,
                                                 double* __restrict__ rinv)
{
    for (int idx = threadIdx.x; idx < NB * NB; idx += NT) {
        const int i = idx >> 6, j = idx & 63;
        const bool in = i < nb && j < nb;
        G[idx] = (in && j <= i) ? Xm[i * DL + j] : 0.0;
        if (in && j >= i) {
            U[(int64_t)(o + i) * ld + o + j] = Am[i * DL + j];
            Un[(int64_t)(o + i) * ld + o + j] = (i == j) ? 1.0 : Am[i * DL + j] * rv[i];
        }
    }
    if (threadIdx.x < NB) rinv[threadIdx.x] = (threadIdx.x < nb) ? rv[threadIdx.x] : 0.0;
}

// Diagonal block of the elimination (stand-alone launch).
//   out: U[o+j, o+j : o+nb]  = pivot row j inside the block
//        Un = U / pivot
//        G (64 x 64, ld 64)  = (Un11^T)^-1: pivot rows right of the block are G * A[o:o+nb, o+nb:];
//        rinv[j] = 1 / pivot_j
__global__ __launch_bounds__(NT) void elim_diag_kernel(const double* __restrict__ A, int64_t ld, int o, int nb,
                                                        double* __restrict__ U, double* __restrict__ Un,
                                                        double* __restrict__ G, double* __restrict__ rinv,
                                                        int* __restrict__ flag)
{
    __shared__ double Am[NB * DL];
    __shared__ double Xm[NB * DL];
    __shared__ double rv[SWEEP_LDS];
    for (int idx = threadIdx.x; idx < NB * NB; idx += NT) {
        const int i = idx >> 6, j = idx & 63;
        double v = (i == j) ? 1.0 : 0.0;
        if (i < nb && j < nb) v = A[(int64_t)(o + min(i, j)) * ld + o + max(i, j)];   // upper triangle is the maintained one
        Am[i * DL + j] = v;
    }
    __syncthreads();
    elim_block(Am, Xm, rv, flag);
    elim_block_store(Am, Xm, rv, ld, o, nb, U, Un, G, rinv);
}

// Shared-Hinv elimination of the first `steps` columns, `block` columns at a time: diagonal block, pivot rows, trailing
// update.  (All columns in blocks of 64: launch_flow_eliminate.)
hipError_t eliminate_blocked(fobq_ctx* c, double* A, int d, int steps, int block, double* U, double* Un, int* flag,
                             const std::vector<hipEvent_t>* rows_ready)
{
    hipStream_t s = c->stream;
    auto ready = [&](int k) {
        if (rows_ready && k < (int)rows_ready->size())
            (void)hipEventRecord((*rows_ready)[k], s);
    };
    double* G = c->Dblk.as<double>();
    double* rinv = G + NB * NB;
    int it = 0;
    for (int o = 0; o < steps; o += block, ++it) {
        const int nb = min(block, steps - o);
        hipLaunchKernelGGL(elim_diag_kernel, dim3(1), dim3(NT), 0, s, A, (int64_t)d, o, nb, U, Un, G, rinv, flag);
        const int r = d - o - nb;
        if (r <= 0) { ready(it); break; }
        // pivot rows right of the block: U12 = G * A12, Un12 = D^-1 U12
        GemmP p;
        p.M = nb; p.N = r; p.K = nb;
        p.A = G; p.lda = NB;
        p.B = A + (int64_t)o * d + (o + nb); p.ldb = d;
        p.C = U + (int64_t)o * d + (o + nb); p.ldc = d;
        p.C2 = Un + (int64_t)o * d + (o + nb); p.rowscale = rinv;
        hipError_t e = gemm64(s, p, false, false);
        if (e != hipSuccess) return e;
        // trailing update  A22 -= Un12^T U12  (tiles on or above the diagonal)
        GemmP q;
        q.M = r; q.N = r; q.K = nb;
        q.A = Un + (int64_t)o * d + (o + nb); q.lda = d;
        q.B = U + (int64_t)o * d + (o + nb); q.ldb = d;
        q.C = A + (int64_t)(o + nb) * d + (o + nb); q.ldc = d;
        q.alpha = -1.0; q.beta = 1.0; q.cmode = CMODE_UPPER;
        e = gemm64(s, q, true, false);
        if (e != hipSuccess) return e;
        ready(it);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Batched small layers (d <= 256, at most 4 panels).  A layer this small never fills the GPU: its whole
// factor path is a chain of dependent steps on one workgroup's worth of work.  Here ONE workgroup per layer
// walks that chain by itself -- blocked with the same 64 x 64 diagonal-block routines, the tile products on
// the matrix cores with operands straight from global memory (everything sits in L2) -- so that a single
// launch factors every layer of a batch, and the launch count no longer grows with the number of layers.
//
// tile_mm: C (m x n) = beta C + alpha op(A) op(B), op(A) m x k, op(B) k x n, all <= 64, row-major in global memory.
//   TA: op(A)[r][q] = A[q * lda + r] (else A[r * lda + q]);  TB: op(B)[q][c] = B[c * ldb + q] (else B[q * ldb + c]).
//   C2 / rowscale (may be null): C2[r][c] = rowscale[r] * result.
// The two operand tiles are staged in LDS as they lie in memory (coalesced rows; Pa, Pb: NB * DL doubles each)
// and the MFMA fragments are read in the orientation the product needs.  Called by all NT threads; every
// operand is in LDS before anything is stored (C may alias A or B); ends with a barrier.
template <bool TA, bool TB>
__device__ __forceinline__ void tile_mm(double* Pa, double* Pb, double* C, int64_t ldc, const double* A, int64_t lda,
                                        const double* B, int64_t ldb, int m, int n, int k, double alpha, double beta,
                                        double* C2 = nullptr, const double* rowscale = nullptr)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
    const int arows = TA ? k : m, acols = TA ? m : k, brows = TB ? n : k, bcols = TB ? k : n;
    double pa[8], pb[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int y = wave + 8 * u, x = lane;
        pa[u] = (y < arows && x < acols) ? A[(int64_t)y * lda + x] : 0.0;
        pb[u] = (y < brows && x < bcols) ? B[(int64_t)y * ldb + x] : 0.0;
    }
    d4 acc[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = wr * 16 + 4 * v + fq, c = w2 * 32 + 16 * j + fr;
            acc[j][v] = (beta != 0.0 && r < m && c < n) ? beta * C[(int64_t)r * ldc + c] : 0.0;
        }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        Pa[(wave + 8 * u) * DL + lane] = alpha * pa[u];
        Pb[(wave + 8 * u) * DL + lane] = pb[u];
    }
    __syncthreads();
    const int ar = wr * 16 + fr;
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
        const int q = 4 * ks + fq;
        const double av = TA ? Pa[q * DL + ar] : Pa[ar * DL + q];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int bc = w2 * 32 + 16 * j + fr;
            acc[j] = mfma4(av, TB ? Pb[bc * DL + q] : Pb[q * DL + bc], acc[j]);
        }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = wr * 16 + 4 * v + fq, c = w2 * 32 + 16 * j + fr;
            if (r < m && c < n) {
                C[(int64_t)r * ldc + c] = acc[j][v];
                if (C2) C2[(int64_t)r * ldc + c] = acc[j][v] * rowscale[r];
            }
        }
    __syncthreads();
}

// Damped Hessian -> Hinv = L^-T L^-1 (upper tiles; Section 5 item 1, Section 6.1), one workgroup per layer.
__global__ __launch_bounds__(NT) void batch_inverse_kernel(const BatchLayer* __restrict__ layers)
{
    __shared__ double Am[NB * DL];
    __shared__ double Xm[NB * DL];
    __shared__ double rq[SWEEP_LDS];
    const BatchLayer L = layers[blockIdx.x];
    const int d = L.d, T = (d + NB - 1) / NB, tid = threadIdx.x;
    // lambda = damp * mean(diag H) + damp_abs; the diagonal is summed in index order by one wavefront-sized tree
    {
        double s = 0.0;
        for (int a = tid; a < d; a += NT) s += L.H[(int64_t)a * d + a];
        Xm[tid] = s;
        __syncthreads();
        for (int w = NT / 2; w > 0; w >>= 1) {
            if (tid < w) Xm[tid] += Xm[tid + w];
            __syncthreads();
        }
    }
    const double lam = L.damp * (Xm[0] / (double)d) + L.damp_abs;
    __syncthreads();
    for (int idx = tid; idx < d * d; idx += NT) {
        const int a = idx / d, b = idx - a * d;
        L.Hd[idx] = L.H[idx] + (a == b ? lam : 0.0);
    }
    __syncthreads();
    // H_d = L L^T, right-looking over the panels; L overwrites the lower tiles of Hd
    for (int p = 0; p < T; ++p) {
        const int o = NB * p, nb = min(NB, d - o);
        for (int idx = tid; idx < NB * NB; idx += NT) {
            const int i = idx >> 6, j = idx & 63;
            double v = (i == j) ? 1.0 : 0.0;                    // identity padding past nb
            if (i < nb && j < nb) v = (j <= i) ? L.Hd[(int64_t)(o + i) * d + o + j] : 0.0;
            Am[i * DL + j] = v;
        }
        __syncthreads();
        chol_block(Am, Xm, rq, L.flags + 0);
        for (int idx = tid; idx < NB * NB; idx += NT) {
            const int i = idx >> 6, j = idx & 63;
            if (i < nb && j < nb) {
                L.Hd[(int64_t)(o + i) * d + o + j] = (j <= i) ? Am[i * DL + j] : 0.0;
                L.Linv[(int64_t)(o + i) * d + o + j] = (j <= i) ? Xm[i * DL + j] : 0.0;
            }
        }
        __syncthreads();
        for (int i = p + 1; i < T; ++i) {        // L_ip = A_ip L_pp^-T
            double* t = L.Hd + (int64_t)(NB * i) * d + o;
            tile_mm<false, true>(Am, Xm, t, d, t, d, L.Linv + (int64_t)o * d + o, d, min(NB, d - NB * i), nb, nb, 1.0, 0.0);
        }
        for (int i = p + 1; i < T; ++i)          // A_ij -= L_ip L_jp^T
            for (int j = p + 1; j <= i; ++j)
                tile_mm<false, true>(Am, Xm, L.Hd + (int64_t)(NB * i) * d + NB * j, d, L.Hd + (int64_t)(NB * i) * d + o, d,
                                     L.Hd + (int64_t)(NB * j) * d + o, d, min(NB, d - NB * i), min(NB, d - NB * j), nb, -1.0, 1.0);
    }
    // L^-1 below the diagonal blocks: X_ij = -X_ii sum_{m=j}^{i-1} L_im X_mj
    for (int j = 0; j < T; ++j)
        for (int i = j + 1; i < T; ++i) {
            const int mi = min(NB, d - NB * i), nj = min(NB, d - NB * j);
            double* t = L.T + (int64_t)(NB * i) * d + NB * j;
            for (int m = j; m < i; ++m)
                tile_mm<false, false>(Am, Xm, t, d, L.Hd + (int64_t)(NB * i) * d + NB * m, d, L.Linv + (int64_t)(NB * m) * d + NB * j, d,
                                      mi, nj, min(NB, d - NB * m), 1.0, m > j ? 1.0 : 0.0);
            tile_mm<false, false>(Am, Xm, L.Linv + (int64_t)(NB * i) * d + NB * j, d, L.Linv + (int64_t)(NB * i) * d + NB * i, d, t, d,
                                  mi, nj, mi, -1.0, 0.0);
        }
    // Hinv = L^-T L^-1, tiles on and above the diagonal: Hinv_ij = sum_{m >= j} X_mi^T X_mj
    for (int i = 0; i < T; ++i)
        for (int j = i; j < T; ++j)
            for (int m = j; m < T; ++m)
                tile_mm<true, false>(Am, Xm, L.Hinv + (int64_t)(NB * i) * d + NB * j, d, L.Linv + (int64_t)(NB * m) * d + NB * i, d,
                                     L.Linv + (int64_t)(NB * m) * d + NB * j, d, min(NB, d - NB * i), min(NB, d - NB * j),
                                     min(NB, d - NB * m), 1.0, m > j ? 1.0 : 0.0);
}

// The shared-Hinv elimination (Eq. 12) of a whole small layer: A = Hinv in processing order (gathered here
// through perm), then panel by panel the diagonal block, the pivot rows right of it, the trailing update.
// Leaves U (pivot rows) and Un = U / pivot, both on and above the diagonal.  One workgroup per layer.
__global__ __launch_bounds__(NT) void batch_eliminate_kernel(const BatchLayer* __restrict__ layers)
{
    __shared__ double Am[NB * DL];
    __shared__ double Xm[NB * DL];
    __shared__ double rv[SWEEP_LDS];
    const BatchLayer L = layers[blockIdx.x];
    const int d = L.d, T = (d + NB - 1) / NB, tid = threadIdx.x;
    for (int idx = tid; idx < d * d; idx += NT) {
        const int a = idx / d, b = idx - a * d;
        const int pa = min(max(L.perm[a], 0), d - 1), pb = min(max(L.perm[b], 0), d - 1);
        L.A[idx] = L.Hinv[(int64_t)min(pa, pb) * d + max(pa, pb)];
    }
    __syncthreads();
    for (int p = 0; p < T; ++p) {
        const int o = NB * p, nb = min(NB, d - o);
        for (int idx = tid; idx < NB * NB; idx += NT) {
            const int i = idx >> 6, j = idx & 63;
            double v = (i == j) ? 1.0 : 0.0;
            if (i < nb && j < nb) v = L.A[(int64_t)(o + min(i, j)) * d + o + max(i, j)];
            Am[i * DL + j] = v;
        }
        __syncthreads();
        elim_block(Am, Xm, rv, L.flags + 1);
        for (int idx = tid; idx < NB * NB; idx += NT) {
            const int i = idx >> 6, j = idx & 63;
            const bool in = i < nb && j < nb;
            L.Gs[idx] = (in && j <= i) ? Xm[i * DL + j] : 0.0;
            if (in && j >= i) {
                L.U[(int64_t)(o + i) * d + o + j] = Am[i * DL + j];
                L.Un[(int64_t)(o + i) * d + o + j] = (i == j) ? 1.0 : Am[i * DL + j] * rv[i];
            }
        }
        if (tid < NB) L.rinv[tid] = (tid < nb) ? rv[tid] : 0.0;
        __syncthreads();
        for (int j = p + 1; j < T; ++j)          // pivot rows right of the block: U_pj = G A_pj, Un_pj = D^-1 U_pj
            tile_mm<false, false>(Am, Xm, L.U + (int64_t)o * d + NB * j, d, L.Gs, NB, L.A + (int64_t)o * d + NB * j, d, nb,
                                  min(NB, d - NB * j), nb, 1.0, 0.0, L.Un + (int64_t)o * d + NB * j, L.rinv);
        for (int i = p + 1; i < T; ++i)          // A_ij -= Un_pi^T U_pj
            for (int j = i; j < T; ++j)
                tile_mm<true, false>(Am, Xm, L.A + (int64_t)(NB * i) * d + NB * j, d, L.Un + (int64_t)o * d + NB * i, d,
                                     L.U + (int64_t)o * d + NB * j, d, min(NB, d - NB * i), min(NB, d - NB * j), nb, -1.0, 1.0);
    }
}

hipError_t launch_batch_inverse(hipStream_t s, const BatchLayer* layers, int n)
{
    hipLaunchKernelGGL(batch_inverse_kernel, dim3(n), dim3(NT), 0, s, layers);
    return hipGetLastError();
}

hipError_t launch_batch_eliminate(hipStream_t s, const BatchLayer* layers, int n)
{
    hipLaunchKernelGGL(batch_eliminate_kernel, dim3(n), dim3(NT), 0, s, layers);
    return hipGetLastError();
}

}  // namespace fobq
