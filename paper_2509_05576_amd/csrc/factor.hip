// Factorizations of the path, fp64, blocked with 64-wide panels (the damped inverse is in flow.hip):
//   eliminate_blocked the shared-Hinv elimination of Eq. 12, B columns at a time, for any B and any number of steps
//                    (flow.hip has the form for all columns at B = 64):
//                    after column t is processed, Hinv -= Hinv[:,t] Hinv[t,:] / Hinv[t,t].
//                    The pivot rows are kept:  U[t, t:]  = Hinv^(t)[t, t:]  and
//                    Un[t, :] = U[t, :] / U[t, t]; the weight compensation of Eq. 9 / 11
//                    for step t is  W[:, k] -= (w_t - q_t) * Un[t, k].
// The 64 x 64 diagonal blocks are handled by one workgroup in LDS (tile_block.h); everything
// else is products on the matrix cores (gemm64).
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
        hipError_t e = gemm64(s, p, false);
        if (e != hipSuccess) return e;
        // trailing update  A22 -= Un12^T U12  (tiles on or above the diagonal)
        GemmP q;
        q.M = r; q.N = r; q.K = nb;
        q.A = Un + (int64_t)o * d + (o + nb); q.lda = d;
        q.B = U + (int64_t)o * d + (o + nb); q.ldb = d;
        q.C = A + (int64_t)(o + nb) * d + (o + nb); q.ldc = d;
        q.alpha = -1.0; q.beta = 1.0; q.upper = true;
        e = gemm64(s, q, true);
        if (e != hipSuccess) return e;
        ready(it);
    }
    return hipGetLastError();
}

}  // namespace fobq
