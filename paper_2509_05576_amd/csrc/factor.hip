// Factorizations of the path, fp64, blocked with 64-wide panels (the damped inverse is in flow.hip):
//   eliminate_blocked the shared-Hinv elimination of Eq. 12, B columns at a time:
//                    after column t is processed, Hinv -= Hinv[:,t] Hinv[t,:] / Hinv[t,t].
//                    The pivot rows are kept:  U[t, t:]  = Hinv^(t)[t, t:]  and
//                    Un[t, :] = U[t, :] / U[t, t]; the weight compensation of Eq. 9 / 11
//                    for step t is  W[:, k] -= (w_t - q_t) * Un[t, k].
//   batch_*          the factor path of many small layers, one workgroup per layer
// The 64 x 64 diagonal blocks are handled by one workgroup in LDS (tile_block.h); everything
// else is a rank-64 update on the matrix cores, fused into the panel launches
// (elim_iter_kernel) or through gemm64.
#include <hip/hip_ext.h>

#include "fobq_internal.h"
#include "tile_block.h"

namespace fobq {

// launches with more tiles than this use the two-workgroups-per-compute-unit variant of the panel kernels
constexpr int DENSE_LAUNCH_TILES = 300;
// launches with at least this many trailing tiles are bound by tile throughput: the panel is stored by a launch of
// its own and every tile does one product instead of three (see the modes below)
constexpr int STORED_PANEL_TILES = 800;
// The workgroup that holds the place beside workgroup 0 (see the modes below) has the index `mate_slot` = the number
// of compute units of the device (the first that many workgroups of a launch go to distinct compute units).
constexpr int MATE_MAX_NAPS = 64;


// Fragment layout of a 64 x 64 block inverse M that the next launch uses as an MFMA operand:
//   F[((w * 16 + ks) * 2 + h) * 64 + lane] = M[w * 32 + h * 16 + (lane & 15)][4 * ks + (lane >> 4)]
// so that the 64 lanes of a wavefront read 512 contiguous bytes per operand element instead of
// 16 scattered 32-byte pieces.  frag_source returns the (row, column) of M stored at F[idx].
__device__ __forceinline__ void frag_source(int idx, int& row, int& col)
{
    const int lane = idx & 63, h = (idx >> 6) & 1, ks = (idx >> 7) & 15, w = idx >> 11;
    row = w * 32 + h * 16 + (lane & 15);
    col = 4 * ks + (lane >> 4);
}

// A 64 x 64 lower-triangular block T in the fragment layout (frag_source) as an MFMA operand: operand tile
// t (of 4; 16 rows of T as A-operand, or 16 columns of T^T as B-operand) only needs the k-steps 0 .. 4 t + 3.
// A wavefront takes the two operand tiles {W, 3 - W}, W = 0 or 1: 20 of 32 (k-step, tile) pairs either way.
// W is a template parameter so that the k-loops below are straight-line code: with a run-time W
// every skipped pair is a branch, and the branches keep the LDS reads of one k-step from being
// issued under the MFMAs of the one before.
template <int W>
__device__ __forceinline__ void tri_frag_load(const double* __restrict__ F, int lane, double (&g)[16][2])
{
    constexpr int t[2] = {W, 3 - W};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            g[ks][j] = (ks <= 4 * t[j] + 3) ? F[(((t[j] >> 1) * 16 + ks) * 2 + (t[j] & 1)) * 64 + lane] : 0.0;
}

// li (+ lj if TWO) += P T^T for the wavefront's 16 rows (from row0) and its two column tiles {W, 3 - W}:
// A-operand rows out of LDS (Pi / Pj, row-major [row][k]), B-operand = g.
template <int W, bool TWO>
__device__ __forceinline__ void tri_right_product(const double* Pi, const double* Pj, const double (&g)[16][2],
                                                  int row0, int fr, int fq, d4 (&li)[2], d4 (&lj)[2])
{
    constexpr int t[2] = {W, 3 - W};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
        const double ai = Pi[(row0 + fr) * DL + 4 * ks + fq];
        double aj = 0.0;
        if (TWO) aj = Pj[(row0 + fr) * DL + 4 * ks + fq];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (ks > 4 * t[j] + 3) continue;
            li[j] = mfma4(ai, g[ks][j], li[j]);
            if (TWO) lj[j] = mfma4(aj, g[ks][j], lj[j]);
        }
    }
}

// ui (+ uj if TWO) += T P for the wavefront's two row tiles {W, 3 - W} and its 16 columns (from col0):
// A-operand = g, B-operand columns out of LDS (Pi / Pj, row-major [k][column]).
template <int W, bool TWO>
__device__ __forceinline__ void tri_left_product(const double* Pi, const double* Pj, const double (&g)[16][2],
                                                 int col0, int fr, int fq, d4 (&ui)[2], d4 (&uj)[2])
{
    constexpr int t[2] = {W, 3 - W};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
        const double bi = Pi[(4 * ks + fq) * DL + col0 + fr];
        double bj = 0.0;
        if (TWO) bj = Pj[(4 * ks + fq) * DL + col0 + fr];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (ks > 4 * t[i] + 3) continue;
            ui[i] = mfma4(g[ks][i], bi, ui[i]);
            if (TWO) uj[i] = mfma4(g[ks][i], bj, uj[i]);
        }
    }
}

// Work split of the fused panel kernels below: NT = 512 threads = 8 wavefronts per 64 x 64 tile, two per
// SIMD.  One wavefront alone issues a v_mfma_f64_16x16x4_f64 only every ~140 cycles (measured: 59 ns per
// instruction per wavefront whatever the number of independent accumulators); two wavefronts on a SIMD
// interleave to the pipe's own rate of one per ~64 cycles.  The products of workgroup 0 are on the critical
// path of the whole factorization, so they are spread over twice the wavefronts a 64 x 64 tile needs.
// Wavefront w: wr = w / 2 is its 16-row slice of the tile, w2 = w % 2 its 32-column half (and the parity
// W of its operand tiles in the triangular products).

// Modes of a panel launch.  PANEL_FUSED: every trailing tile recomputes the two panel blocks it needs (three rank-64 products
// per tile instead of one, in exchange for not waiting on a separate panel launch), and workgroup 0 goes on to the next
// diagonal block.  For launches so large that tile throughput bounds them: PANEL_ONLY stores the panel, PANEL_STORED takes it.
// Two such panels can share one pass over the trailing matrix: after the first only the next panel's tiles are updated
// (PANEL_NEAR), after the second every trailing tile takes both panels (PANEL_STORED2), the older one first.
// Two workgroups fit a compute unit with WPS = 4, and the one that lands beside workgroup 0 takes matrix-pipe and LDS time
// from the launch's critical path.  The first 256 workgroups go to distinct compute units, so that neighbour is workgroup
// `mate_slot`; it is not a tile: one of its wavefronts sleeps, holding the place, until workgroup 0 says that it is done
// (mate_flag reaches this launch's epoch) or MATE_MAX_NAPS naps of about 0.4 us have passed.
enum { PANEL_FUSED = 0, PANEL_ONLY = 1, PANEL_STORED = 2, PANEL_NEAR = 3, PANEL_STORED2 = 4 };

__device__ __forceinline__ void elim_block_store(const double* Am, const double* Xm, const double* rv,
                                                 int64_t ld, int o, int nb, double* __restrict__ U,
                                                 double* __restrict__ Un, double* __restrict__ G,
                                                 double* __restrict__ Gf, double* __restrict__ rinv)
{
    for (int idx = threadIdx.x; idx < NB * NB; idx += NT) {
        const int i = idx >> 6, j = idx & 63;
        const bool in = i < nb && j < nb;
        if (G) G[idx] = (in && j <= i) ? Xm[i * DL + j] : 0.0;
        if (Gf) {
            int fi, fj;
            frag_source(idx, fi, fj);
            Gf[idx] = (fi < nb && fj <= fi) ? Xm[fi * DL + fj] : 0.0;
        }
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
//        Gf = the same in the fragment layout (either may be null)
//        rinv[j] = 1 / pivot_j
__global__ __launch_bounds__(NT) void elim_diag_kernel(const double* __restrict__ A, int64_t ld, int o, int nb,
                                                        double* __restrict__ U, double* __restrict__ Un,
                                                        double* __restrict__ G, double* __restrict__ Gf,
                                                        double* __restrict__ rinv, int* __restrict__ flag)
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
    elim_block_store(Am, Xm, rv, ld, o, nb, U, Un, G, Gf, rinv);
}

// One whole iteration of the blocked shared-Hinv elimination in a single launch.  The panel is the 64 rows/columns o .. o+63 whose diagonal block has
// been eliminated (G in the fragment layout, rinv).  Workgroup (ti, tj), ti <= tj, owns tile (ti, tj) of the trailing
// matrix (upper triangle):
//   1. pivot rows right of the block for its two tile columns: U12_i = G A12_i, U12_j, and
//      Un12 = D^-1 U12; the tiles of the first tile row also store them into U and Un;
//   2. A22(ti, tj) -= Un12_i^T U12_j        (Eq. 12 for the 64 columns of the panel at once);
//   3. workgroup 0 eliminates tile (0, 0), the next diagonal block, right away.
// MODE: PANEL_ONLY = workgroup j computes and stores the pivot rows U12_j, Un12_j right of the
// block for its tile column; PANEL_STORED = the trailing launch that follows and takes them from U and Un;
// PANEL_NEAR = only the tiles (0, j) of the next panel's rows, each recomputing and storing its pivot rows;
// PANEL_STORED2 = the 128 pivot rows o - 64 .. o + 63 at once.
template <int WPS, int MODE>
__global__ __launch_bounds__(NT, WPS) void elim_iter_kernel(double* __restrict__ A, int d, int o,
                                                       const double* __restrict__ G, const double* __restrict__ rinv,
                                                       double* __restrict__ U, double* __restrict__ Un,
                                                       double* __restrict__ G_next, double* __restrict__ rinv_next,
                                                       int* __restrict__ flag, int* __restrict__ mate_flag, int epoch, int mate_slot)
{
    __shared__ double lds[SWEEP_LDS + 2 * NB * DL];   // sweep scratch, two tiles: 2 workgroups per compute unit
    // epoch != 0: the launch has one workgroup more than tiles, and workgroup `mate_slot` only holds the place
    // beside workgroup 0 (see above; both variants of this kernel fit two workgroups per compute unit)
    if (epoch != 0 && (int)blockIdx.x == mate_slot) {
        if (threadIdx.x >= 64) return;
        for (int i = 0; i < MATE_MAX_NAPS; ++i) {
            if (__hip_atomic_load(mate_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - epoch >= 0) break;
            __builtin_amdgcn_s_sleep(16);
        }
        return;
    }
    const int bid = (int)blockIdx.x - ((epoch != 0 && (int)blockIdx.x > mate_slot) ? 1 : 0);
    double* Pi = lds + SWEEP_LDS;
    double* Pj = Pi + NB * DL;
    double* rs = lds;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
    const int r0 = o + NB;
    int ti, tj;
    if (MODE == PANEL_ONLY) { ti = bid; tj = bid; }      // workgroup j: tile column j of the pivot rows
    else if (MODE == PANEL_NEAR) { ti = 0; tj = bid; }   // workgroup j: tile (0, j), the rows of the next panel
    else tri_decode(bid, tj, ti);     // ti <= tj
    const bool diag_tile = ti == tj;
    const int ci0 = r0 + NB * ti, cj0 = r0 + NB * tj;
    constexpr bool STORED = MODE == PANEL_STORED || MODE == PANEL_STORED2;

    d4 c[2];
    if (STORED) {
        // Un12_i and U12_j as the panel launch(es) stored them; the trailing tile itself in flight meanwhile
        const int o1 = MODE == PANEL_STORED2 ? o - NB : o;      // the panel that is applied first
        double pa[8], pb[8], qa[8], qb[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int y = wave + 8 * u, x = lane;
            pa[u] = Un[(int64_t)(o1 + y) * d + min(ci0 + x, d - 1)];
            pb[u] = U[(int64_t)(o1 + y) * d + min(cj0 + x, d - 1)];
        }
        if (MODE == PANEL_STORED2) {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int y = wave + 8 * u, x = lane;
                qa[u] = Un[(int64_t)(o + y) * d + min(ci0 + x, d - 1)];
                qb[u] = U[(int64_t)(o + y) * d + min(cj0 + x, d - 1)];
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gm = ci0 + wr * 16 + 4 * v + fq, gn = cj0 + w2 * 32 + j * 16 + fr;
                c[j][v] = A[(int64_t)min(gm, d - 1) * d + min(gn, d - 1)];
            }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int y = wave + 8 * u, x = lane;
            Pi[y * DL + x] = pa[u];
            Pj[y * DL + x] = pb[u];
        }
        __syncthreads();
        if (MODE == PANEL_STORED2) {
            // the older panel's product here, then the newer panel takes its place in LDS for the product below
#pragma unroll
            for (int ks = 0; ks < 16; ++ks) {
                const double a = -Pi[(4 * ks + fq) * DL + wr * 16 + fr];
#pragma unroll
                for (int j = 0; j < 2; ++j) c[j] = mfma4(a, Pj[(4 * ks + fq) * DL + w2 * 32 + j * 16 + fr], c[j]);
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int y = wave + 8 * u, x = lane;
                Pi[y * DL + x] = qa[u];
                Pj[y * DL + x] = qb[u];
            }
            __syncthreads();
        }
    } else {
    // Pivot rows U12 = G A12: G is lower triangular, so the 16 rows of row tile rt (of 4) only need
    // the k-steps 0 .. 4 rt + 3.  The wavefronts with w2 = 0 take the row tiles 0 and 3, those with
    // w2 = 1 the tiles 1 and 2 (20 of 32 (k-step, tile) pairs each), for the 16 columns of slice wr.
    const int rt[2] = {w2, 3 - w2};
    // this lane's A-operand elements of G for those k-steps, straight from global memory
    double ga[16][2];
    if (w2 == 0) tri_frag_load<0>(G, lane, ga); else tri_frag_load<1>(G, lane, ga);
    // one round of loads (all in flight together), then the stores to LDS
    double pa[8], pb[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int y = wave + 8 * u, x = lane;
        // Columns past d are read from column d - 1 (clamped address, no branch per load): they
        // only reach outputs past d, which are never stored or are replaced by the identity padding.
        pa[u] = A[(int64_t)(o + y) * d + min(ci0 + x, d - 1)];
    }
    if (!diag_tile) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int y = wave + 8 * u, x = lane;
            pb[u] = A[(int64_t)(o + y) * d + min(cj0 + x, d - 1)];
        }
    }
    const double rsv = (tid < NB) ? rinv[tid] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int y = wave + 8 * u, x = lane;
        Pi[y * DL + x] = pa[u];
        if (!diag_tile) Pj[y * DL + x] = pb[u];
    }
    if (tid < NB) rs[tid] = rsv;
    __syncthreads();
    // the trailing tile itself (rows of slice wr, the 32 columns of half w2): in flight during the product
    if (MODE == PANEL_FUSED || MODE == PANEL_NEAR) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gm = ci0 + wr * 16 + 4 * v + fq, gn = cj0 + w2 * 32 + j * 16 + fr;
                c[j][v] = A[(int64_t)min(gm, d - 1) * d + min(gn, d - 1)];
            }
    }

    d4 ui[2], uj[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) { ui[i] = d4{0.0, 0.0, 0.0, 0.0}; uj[i] = d4{0.0, 0.0, 0.0, 0.0}; }
    if (w2 == 0) {
        if (diag_tile) tri_left_product<0, false>(Pi, Pj, ga, wr * 16, fr, fq, ui, uj);
        else tri_left_product<0, true>(Pi, Pj, ga, wr * 16, fr, fq, ui, uj);
    } else {
        if (diag_tile) tri_left_product<1, false>(Pi, Pj, ga, wr * 16, fr, fq, ui, uj);
        else tri_left_product<1, true>(Pi, Pj, ga, wr * 16, fr, fq, ui, uj);
    }
    __syncthreads();
    // Pi := Un12_i (rows scaled by 1 / pivot), Pj := U12_j
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int m = rt[i] * 16 + 4 * v + fq, n = wr * 16 + fr;
            const double uiv = ui[i][v];
            const double ujv = diag_tile ? uiv : uj[i][v];
            Pi[m * DL + n] = uiv * rs[m];
            Pj[m * DL + n] = ujv;
            if ((ti == 0 || MODE == PANEL_ONLY) && cj0 + n < d) {
                U[(int64_t)(o + m) * d + cj0 + n] = ujv;
                Un[(int64_t)(o + m) * d + cj0 + n] = ujv * rs[m];
            }
        }
    if (MODE == PANEL_ONLY) return;
    __syncthreads();
    }
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
        const double a = -Pi[(4 * ks + fq) * DL + wr * 16 + fr];
#pragma unroll
        for (int j = 0; j < 2; ++j) c[j] = mfma4(a, Pj[(4 * ks + fq) * DL + w2 * 32 + j * 16 + fr], c[j]);
    }
    if (bid != 0) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gm = ci0 + wr * 16 + 4 * v + fq, gn = cj0 + w2 * 32 + j * 16 + fr;
                if (gm < d && gn < d) A[(int64_t)gm * d + gn] = c[j][v];
            }
        return;
    }
    // tile (0, 0): the next diagonal block, of size nbn
    const int nbn = min(NB, d - r0);
    __syncthreads();
    double* Am = Pi;
    double* Xm = Pj;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int m = wr * 16 + 4 * v + fq, n = w2 * 32 + j * 16 + fr;
            Am[m * DL + n] = (m < nbn && n < nbn) ? c[j][v] : (m == n ? 1.0 : 0.0);
        }
    __syncthreads();
    elim_block(Am, Xm, rs, flag);
    elim_block_store(Am, Xm, rs, d, r0, nbn, U, Un, nullptr, G_next, rinv_next);
    if (epoch != 0 && threadIdx.x == 0) __hip_atomic_store(mate_flag, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Shared-Hinv elimination of the first `steps` columns, `block` columns at a time.
hipError_t eliminate_blocked(fobq_ctx* c, double* A, int d, int steps, int block, double* U, double* Un, int* flag,
                             const std::vector<hipEvent_t>* rows_ready)
{
    hipStream_t s = c->stream;
    auto ready = [&](int k) {
        if (rows_ready && k < (int)rows_ready->size())
            (void)hipEventRecord((*rows_ready)[k], s);
    };
    double* Gb[2] = {c->Dblk.as<double>() + 2 * NB * NB, c->Dblk.as<double>() + 3 * NB * NB};
    double* rb[2] = {c->Dblk.as<double>() + 4 * NB * NB, c->Dblk.as<double>() + 4 * NB * NB + NB};
    if (block == NB && steps == d) {
        // one stand-alone launch for the first diagonal block, then one fused launch per panel
        hipLaunchKernelGGL(elim_diag_kernel, dim3(1), dim3(NT), 0, s, A, (int64_t)d, 0, min(NB, d), U, Un,
                           (double*)nullptr, Gb[0], rb[0], flag);
        int it = 0;
        for (int o = 0; o + NB < d; o += NB, ++it) {
            const int T = (d - o - NB + NB - 1) / NB;
            // rows of block `it` are complete when this launch is (its diagonal part came from the previous
            // one): the block's event rides on the launch itself as its stop event -- a separate
            // hipEventRecord between two dependent launches costs about 4 us of bubble
            hipEvent_t done = (rows_ready && it < (int)rows_ready->size()) ? (*rows_ready)[it] : nullptr;
            const int tiles = T * (T + 1) / 2;
            // a launch with a workgroup of index `cus` gets one more, which holds the place beside workgroup 0
            const bool mate = tiles > c->cus;
            const int epoch = mate ? ++c->mate_epoch : 0;
            int* mate_flag = c->flags.as<int>() + FLAG_WORD_MATE;
            if (tiles >= STORED_PANEL_TILES) {
                const int T2 = T - 1, tiles2 = T2 * (T2 + 1) / 2;
                if (tiles2 >= STORED_PANEL_TILES) {
                    // two panels, one pass over the trailing matrix (see the modes below): the next panel's rows now,
                    // both panels' update of everything else after the next panel
                    hipExtLaunchKernelGGL((elim_iter_kernel<2, PANEL_NEAR>), dim3(T), dim3(NT), 0, s, nullptr, done, 0, A, d, o,
                                          (const double*)Gb[it & 1], (const double*)rb[it & 1], U, Un, Gb[(it + 1) & 1],
                                          rb[(it + 1) & 1], flag, mate_flag, 0, c->cus);
                    o += NB;
                    ++it;
                    hipEvent_t done2 = (rows_ready && it < (int)rows_ready->size()) ? (*rows_ready)[it] : nullptr;
                    hipLaunchKernelGGL((elim_iter_kernel<2, PANEL_ONLY>), dim3(T2), dim3(NT), 0, s, A, d, o,
                                       (const double*)Gb[it & 1], (const double*)rb[it & 1], U, Un, Gb[(it + 1) & 1],
                                       rb[(it + 1) & 1], flag, mate_flag, 0, c->cus);
                    hipExtLaunchKernelGGL((elim_iter_kernel<4, PANEL_STORED2>), dim3(tiles2 + 1), dim3(NT), 0, s, nullptr, done2, 0,
                                          A, d, o, (const double*)Gb[it & 1], (const double*)rb[it & 1], U, Un, Gb[(it + 1) & 1],
                                          rb[(it + 1) & 1], flag, mate_flag, ++c->mate_epoch, c->cus);
                } else {
                    // throughput-bound launch: the pivot rows once (T workgroups), then one product per trailing tile
                    hipLaunchKernelGGL((elim_iter_kernel<2, PANEL_ONLY>), dim3(T), dim3(NT), 0, s, A, d, o,
                                       (const double*)Gb[it & 1], (const double*)rb[it & 1], U, Un, Gb[(it + 1) & 1],
                                       rb[(it + 1) & 1], flag, mate_flag, 0, c->cus);
                    hipExtLaunchKernelGGL((elim_iter_kernel<4, PANEL_STORED>), dim3(tiles + 1), dim3(NT), 0, s, nullptr, done, 0, A,
                                          d, o, (const double*)Gb[it & 1], (const double*)rb[it & 1], U, Un, Gb[(it + 1) & 1],
                                          rb[(it + 1) & 1], flag, mate_flag, epoch, c->cus);
                }
            } else if (tiles <= DENSE_LAUNCH_TILES)
                hipExtLaunchKernelGGL((elim_iter_kernel<2, PANEL_FUSED>), dim3(tiles + (mate ? 1 : 0)), dim3(NT), 0, s, nullptr, done, 0, A,
                                      d, o, (const double*)Gb[it & 1], (const double*)rb[it & 1], U, Un, Gb[(it + 1) & 1],
                                      rb[(it + 1) & 1], flag, mate_flag, epoch, c->cus);
            else
                hipExtLaunchKernelGGL((elim_iter_kernel<4, PANEL_FUSED>), dim3(tiles + (mate ? 1 : 0)), dim3(NT), 0, s, nullptr, done, 0, A,
                                      d, o, (const double*)Gb[it & 1], (const double*)rb[it & 1], U, Un, Gb[(it + 1) & 1],
                                      rb[(it + 1) & 1], flag, mate_flag, epoch, c->cus);
        }
        ready(it);              // last block: only a diagonal part
        return hipGetLastError();
    }
    // general form (any block width, partial elimination): diagonal block, pivot rows, trailing update
    double* G = Gb[0];
    double* rinv = rb[0];
    int it = 0;
    for (int o = 0; o < steps; o += block, ++it) {
        const int nb = min(block, steps - o);
        hipLaunchKernelGGL(elim_diag_kernel, dim3(1), dim3(NT), 0, s, A, (int64_t)d, o, nb, U, Un, G,
                           (double*)nullptr, rinv, flag);
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
