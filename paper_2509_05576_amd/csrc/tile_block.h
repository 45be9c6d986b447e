// 64 x 64 diagonal blocks of the factorizations, held in LDS by one workgroup (device code shared by factor.hip and
// flow.hip).
#pragma once
#include "fobq_internal.h"

namespace fobq {

constexpr int NB = 64;

// ---------------------------------------------------------------------------
// 64 x 64 diagonal blocks.  Both diagonal-block kernels keep the block in LDS and
// work on it as a 4 x 4 grid of 16 x 16 tiles.  The only sequential arithmetic is
// the unblocked sweep over the 16 pivots of a diagonal tile: one wavefront, one
// row (Cholesky) or column (elimination) of the whole block per lane, so the same
// sweep also produces the tiles below (right of) the diagonal tile; pivot rows are
// broadcast with v_readlane (next column) and LDS reads (the columns after it).  A
// wavefront on its own issues one instruction of any kind per 5 to 8 cycles, so the
// sweep costs its instruction count.  The triangular inverse of a diagonal tile comes out
// of the same sweep, in lanes it would leave idle (the first tile's: a forward
// substitution on a second wavefront during the next sweep).  Everything else --
// trailing update, assembly of the 64 x 64 triangular inverse from the tile
// inverses -- is 16 x 16 x 16 products on the matrix cores (4 MFMAs each), one tile
// per wavefront, one interval behind the sweeps.
typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int NT = 512;   // threads per workgroup of every kernel that uses these routines (8 wavefronts)
constexpr int DL = 66;    // LDS row stride (doubles): conflict-free 8-byte MFMA fragment reads per half-wave
constexpr int CB0 = 48, CB_LEN = CB0 + 16 * 16 + 48;   // sweep column buffer: see chol_block
constexpr int SWEEP_LDS = NB + CB_LEN + 16 * DL;   // doubles of LDS that chol_block / elim_block need besides the two tiles

__device__ __forceinline__ double readlane_f64(double v, int lane)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
    return __hiloint2double(hi, lo);
}

// Reciprocal and reciprocal square root of a pivot (a normal, positive number): the hardware
// approximation r0 (good to about 2^-24) with one third-order correction,
//   1/x       = r0 (1 + e + e^2 + ...),            e = 1 - x r0
//   1/sqrt(x) = y0 (1 + e/2 + 3 e^2 / 8 + ...),    e = 1 - x y0^2
// accurate to about one ulp (measured 1.00 / 1.24 ulp, the same as two Newton steps).  Four / five
// dependent operations: these sit on the sequential path of the tile sweeps.
__device__ __forceinline__ double pivot_rcp(double x)
{
    const double r0 = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, r0, 1.0);
    return fma(r0 * e, 1.0 + e, r0);
}

__device__ __forceinline__ double pivot_rsqrt(double x)
{
    const double y0 = __builtin_amdgcn_rsq(x);
    const double e = fma(-(x * y0), y0, 1.0);
    return fma(y0 * e, fma(0.375, e, 0.5), y0);
}

// The same value, which the compiler computes where it stands and does not know: keeps lane-dependent constants from being
// prepared ahead of a loop (and spilled), and LDS offsets as one register plus an immediate.
__device__ __forceinline__ int here(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}

__device__ __forceinline__ d4 mfma4(double a, double b, d4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// One off-diagonal 16 x 16 tile of the inverse X of a 64 x 64 lower triangular matrix T:
//   X_ij = -X_ii sum_{m=j}^{i-1} T_im X_mj        (X_ii and the X_mj already in Xm).
// tfetch(i, m, ks) returns this lane's A-operand element of tile T_im for k-step ks, i.e.
// T_im[fr][4 ks + fq].  One wavefront.  inv_tile_sum adds the terms m0 <= m < m1 to t,
// inv_tile_finish multiplies by -X_ii and stores the tile.
template <class TF>
__device__ __forceinline__ d4 inv_tile_sum(const double* Xm, TF tfetch, int i, int j, int m0, int m1, d4 t, int fr,
                                           int fq)
{
    for (int m = m0; m < m1; ++m)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            t = mfma4(tfetch(i, m, ks), Xm[(16 * m + 4 * ks + fq) * DL + 16 * j + fr], t);
    return t;
}

__device__ __forceinline__ void inv_tile_finish(double* Xm, int i, int j, d4 t, int fr, int fq)
{
    // the accumulator layout (row 4 v + fq, column fr) is the B-operand layout of k-step v
    d4 r = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) r = mfma4(Xm[(16 * i + fr) * DL + 16 * i + 4 * ks + fq], t[ks], r);
#pragma unroll
    for (int v = 0; v < 4; ++v) Xm[(16 * i + 4 * v + fq) * DL + 16 * j + fr] = -r[v];
    __builtin_amdgcn_wave_barrier();
}

template <class TF>
__device__ __forceinline__ void inv_tile(double* Xm, TF tfetch, int i, int j, int fr, int fq)
{
    inv_tile_finish(Xm, i, j, inv_tile_sum(Xm, tfetch, i, j, j, i, d4{0.0, 0.0, 0.0, 0.0}, fr, fq), fr, fq);
}

// Schedule shared by chol_block and elim_block.  sweep(b): pivots of diagonal tile b and the
// tiles below / right of it -- and, for b >= 1, the inverse X_bb of the diagonal tile, carried along in
// 16 lanes that the sweep leaves idle; tinv(0): triangular inverse of diagonal tile 0 into Xm;
// trail(b): update of the tiles behind tile row/column b; tf: tile fetch for inv_tile.
//   interval   wavefront 0        wavefront 1   wavefront 2   wavefronts 3, 4, 5
//   b = 0      sweep(0)
//   b = 1      sweep(1) + X_11    tinv(0)
//   b = 2      sweep(2) + X_22                  X_10
//   b = 3      sweep(3) + X_33    X_21          X_20          the sums of X_30, X_31, X_32 as far as they
//                                                             do not need this interval's tiles
//   then                                                      rest of the sums, times -X_33
//   (after each of b = 0..2: trail(b) on all wavefronts)
// Called by all NT threads of the workgroup (at least 6 wavefronts); ends with a barrier.
// `beside` is called by wavefronts 1 .. 7 during the first sweep: the caller's work on tiles of the block that this sweep does
// not read (it reads the first tile column / row only; the diagonal entries of later tiles that its lanes carry along are not
// used).  `ahead` is called by every wavefront about 2 us before the end (wavefront 0: after the last sweep).
struct Nothing { __device__ void operator()() const {} };
template <class SW, class TI, class TR, class TF, class BS, class AH>
__device__ __forceinline__ void block_schedule(double* Xm, SW sweep, TI tinv, TR trail, TF tf, BS beside, AH ahead)
{
    const int lane = here(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int fr = lane & 15, fq = lane >> 4;
    d4 t = {0.0, 0.0, 0.0, 0.0};
    const int j3 = wave - 3;                       // wavefronts 3, 4, 5: column tile of X_3j
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if (b == 3 && wave != 0) ahead();
        if (wave == 0) sweep(b);
        else if (b == 0) beside();
        else if (wave == 1 && b == 1) tinv(0);
        else if (wave == 2 && b == 2) inv_tile(Xm, tf, 1, 0, fr, fq);
        else if (wave == 1 && b == 3) inv_tile(Xm, tf, 2, 1, fr, fq);
        else if (wave == 2 && b == 3) inv_tile(Xm, tf, 2, 0, fr, fq);
        else if (wave >= 3 && wave <= 5 && b == 3)
            t = inv_tile_sum(Xm, tf, 3, j3, j3, j3 == 2 ? 3 : 2, t, fr, fq);   // X_2j is not there yet
        if (b == 3 && wave == 0) ahead();
        __syncthreads();
        if (b < 3) {
            trail(b);
            __syncthreads();
        }
    }
    if (wave >= 3 && wave <= 5) {
        if (j3 < 2) t = inv_tile_sum(Xm, tf, 3, j3, 2, 3, t, fr, fq);
        inv_tile_finish(Xm, 3, j3, t, fr, fq);
    }
    __syncthreads();
}

// Cholesky of the 64 x 64 block held in LDS.
//   in : Am lower triangle = the block (identity padding past its size); Xm need not be initialised (every
//        entry of its lower triangle, whole diagonal 16 x 16 tiles included, is written before it is read)
//   out: Am = L (lower; what is above the diagonal is not defined),
//        Xm = L^-1 (lower);  rq (SWEEP_LDS doubles of LDS) is scratch: 1 / L[k][k], then the sweep columns
//   flag: set to 1 when a pivot is <= 0 or not finite (the pivot is replaced by 1 so that
//         the arithmetic stays finite; the caller reports ENOTPD).
// Called by all NT threads of the workgroup; ends with a barrier.
template <class BS = Nothing, class AH = Nothing>
__device__ __forceinline__ void chol_block(double* Am, double* Xm, double* rq, int* __restrict__ flag, BS beside = BS(), AH ahead = AH())
{
    const int tid = here(threadIdx.x), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 15, fq = lane >> 4;
    // The columns of the running sweep: column k at cb[CB0 + 16 k + r], r = row - tile base.  Only the
    // 16 tile rows are read; what the other lanes write falls into the slots of neighbouring columns,
    // which is harmless: a column is read right after it is written, before the next one is written.
    double* cb = rq + NB;
    double* idt = cb + CB_LEN; // 16 rows of the identity, row stride DL (read from the second sweep on)
    if (tid < 256) idt[(tid >> 4) * DL + (tid & 15)] = (tid >> 4) == (tid & 15) ? 1.0 : 0.0;

    // Right-looking Cholesky of the 16 columns base .. base+15 of the block over all rows
    // >= base: lane rho holds row rho.  Rows inside the diagonal tile (0 <= r < 16) hold the
    // tile row (what lies right of its diagonal is carried along and never used); rows below it
    // (r >= 16) get their part of L in the same sweep (l_rho,k = (a_rho,k - sum l l) / l_kk);
    // rows above (r < 0) idle on harmless values.
    auto sweep = [&](int b) {
        const int base = 16 * b, rho = lane, r = rho - base;
        // For b >= 1 the lanes 0..15 (rows above the tile, otherwise idle) carry the rows of the identity
        // as if they were rows below the tile: those become I L_bb^-T, i.e. lane c ends with column c of
        // X_bb = L_bb^-1, for the price of no extra instruction.
        const bool idl = b > 0 && lane < 16;
        // one row of 16 per lane: its own (columns j > r of a tile row are never used), or a row of the identity
        const double* src = idl ? idt + lane * DL : Am + rho * DL + base;
        double a[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) a[j] = src[j];
        // Each lane of the tile also keeps its own diagonal entry in `dg` and updates it locally
        // (dg -= l_rk^2), so the pivot of step k+1 is available one fma after l_rk: the
        // sequential chain per step is readlane, reciprocal square root, multiply, fma.  A wavefront on
        // its own issues an instruction of any kind every 5 to 8 cycles, so the sweep costs its
        // instruction count: nothing sits in the loop that can be done once after it.
        double dg = Am[rho * DL + rho];
        double tp = 0.0, lb[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const double rs = pivot_rsqrt(readlane_f64(dg, base + k));     // 1 / L[k][k]
            // l_rk for r >= k (lane k's a[k] has had the same updates as its dg: it is the pivot).  Lanes
            // of rows above the pivot go through the same arithmetic on entries that are never stored.
            const double t = a[k] * rs;
            dg -= t * t;
            a[k] = t;
            // Rank-1 update of the columns behind: the next column takes l_jk by readlane (it is on the
            // sequential path), the others take it one step late as a broadcast read of the column that
            // every lane leaves in LDS: half an instruction per column instead of two readlanes.
            cb[CB0 + 16 * k + r] = t;
            if (k > 0) {
#pragma unroll
                for (int j = k + 1; j < 16; ++j) a[j] -= tp * lb[j];
            }
            if (k < 15) a[k + 1] -= t * readlane_f64(t, base + k + 1);
#pragma unroll
            for (int j = k + 2; j < 16; ++j) lb[j] = cb[CB0 + 16 * k + j];   // in flight during the next pivot
            tp = t;
        }
        if (r >= 0) {
#pragma unroll
            for (int j = 0; j < 16; ++j) Am[rho * DL + base + j] = a[j];
            if (r < 16) {
                // A pivot that is not a positive normal number (nor anything after it) leaves no positive
                // finite L[r][r] behind: one test per tile row after the sweep instead of one per pivot.
                const double lrr = Am[rho * DL + rho];
                if (!(lrr > 0.0) || !(lrr < 1.0e300)) *flag = 1;
                rq[rho] = pivot_rcp(lrr);
            }
        }
        if (idl) {
#pragma unroll
            for (int k = 0; k < 16; ++k) Xm[(base + k) * DL + base + lane] = a[k];
        }
    };
    // the diagonal tile's inverse by forward substitution: lane c (mod 16) solves L x = e_c;
    // the entries of L and the pivot reciprocals are wavefront-uniform LDS reads
    auto tinv = [&](int b) {
        const int base = 16 * b, c = here(fr);
        double sv[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) sv[i] = (i == c) ? 1.0 : 0.0;
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const double xm = sv[m] * rq[base + m];
            sv[m] = xm;
#pragma unroll
            for (int i = m + 1; i < 16; ++i) sv[i] -= Am[(base + i) * DL + base + m] * xm;
        }
        if (lane < 16) {
#pragma unroll
            for (int i = 0; i < 16; ++i) Xm[(base + i) * DL + base + c] = sv[i];
        }
        __builtin_amdgcn_wave_barrier();
    };
    // trailing tiles: A_ij -= L_ib L_jb^T for b < j <= i
    auto trail = [&](int b) {
        const int base = 16 * b;
        int t = 0;
        for (int i = b + 1; i < 4; ++i)
            for (int j = b + 1; j <= i; ++j, ++t) {
                if ((t & (NT / 64 - 1)) != wave) continue;
                d4 acc;
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[v] = Am[(16 * i + 4 * v + fq) * DL + 16 * j + fr];
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    acc = mfma4(-Am[(16 * i + fr) * DL + base + 4 * ks + fq], Am[(16 * j + fr) * DL + base + 4 * ks + fq], acc);
#pragma unroll
                for (int v = 0; v < 4; ++v) Am[(16 * i + 4 * v + fq) * DL + 16 * j + fr] = acc[v];
            }
    };
    block_schedule(Xm, sweep, tinv, trail,
                   [&](int i, int m, int ks) { return Am[(16 * i + fr) * DL + 16 * m + 4 * ks + fq]; }, beside, ahead);
}

// ---------------------------------------------------------------------------
// Shared-Hinv elimination (Eq. 12) of the 64 x 64 block held in LDS.  With A11 the block,
// U11 its pivot rows, D = diag(U11) and Un11 = D^-1 U11 (unit upper):  A11 = Un11^T D Un11.
//   in : Am upper triangle = the block (identity padding past its size; what is below the diagonal is
//        not used); Xm need not be initialised
//   out: Am upper triangle = U11 (pivot row j = row j; below the diagonal: not defined), rv[j] = 1 / pivot_j
//        (so Un11[i][j] = Am[i][j] * rv[i]),  Xm = G = (Un11^T)^-1 (unit lower)
// Called by all NT threads of the workgroup; ends with a barrier.
template <class BS = Nothing, class AH = Nothing>
__device__ __forceinline__ void elim_block(double* Am, double* Xm, double* rv, int* __restrict__ flag, BS beside = BS(), AH ahead = AH())
{
    const int tid = here(threadIdx.x), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 15, fq = lane >> 4;
    double* cb = rv + NB;      // the pivot rows of the running sweep, laid out as in chol_block
    double* idt = cb + CB_LEN; // 16 rows of the identity, row stride DL (read from the second sweep on)
    if (tid < 256) idt[(tid >> 4) * DL + (tid & 15)] = (tid >> 4) == (tid & 15) ? 1.0 : 0.0;

    // Elimination of the 16 pivots base .. base+15 over all columns >= base: lane c holds
    // column c of the 16 pivot rows.  Columns inside the diagonal tile (0 <= r < 16) hold the
    // tile column (what lies below its diagonal is carried along and never used); columns right
    // of it (r >= 16) get their part of the pivot rows
    // in the same sweep; columns left of it (r < 0) idle on harmless values.
    auto sweep = [&](int b) {
        const int base = 16 * b, c = lane, r = c - base;
        // For b >= 1 the lanes 0..15 (columns left of the tile, otherwise idle) carry the columns of the
        // identity as if they were columns right of the tile: those become G_bb I, i.e. lane c ends with
        // column c of G_bb = (Un_bb^T)^-1.
        const bool idl = b > 0 && lane < 16;
        // one column of 16 per lane: its own (rows j > r of a tile column are never used), or one of the identity
        const double* src = idl ? idt + lane : Am + base * DL + c;
        double a[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) a[j] = src[j * DL];
        // as in chol_block: every lane of the tile keeps its own diagonal entry in `dg`
        double dg = Am[c * DL + c];
        double fp = 0.0, lb[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const double pi = pivot_rcp(readlane_f64(dg, base + k));
            // A[k][c] = U[k][c] for c >= k (lane k's a[k] has had the same updates as its dg: it is the
            // pivot).  Lanes of columns left of the pivot go through the same arithmetic on entries that
            // are never stored.
            const double cr = a[k];
            const double fm = cr * pi;                        // Un[k][c]
            dg -= fm * cr;
            // as in chol_block: the next row by readlane, the others one step late from LDS
            cb[CB0 + 16 * k + r] = cr;
            if (k > 0) {
#pragma unroll
                for (int j = k + 1; j < 16; ++j) a[j] -= fp * lb[j];
            }
            if (k < 15) a[k + 1] -= fm * readlane_f64(cr, base + k + 1);
#pragma unroll
            for (int j = k + 2; j < 16; ++j) lb[j] = cb[CB0 + 16 * k + j];   // in flight during the next pivot
            fp = fm;
        }
        if (r >= 0) {
#pragma unroll
            for (int k = 0; k < 16; ++k) Am[(base + k) * DL + c] = a[k];   // U[k][c] for k <= c
            if (r < 16) {
                // a pivot that is not a positive normal number leaves such a value, or a NaN, on the diagonal
                const double piv = Am[c * DL + c];
                if (!(piv > 0.0) || !(piv < 1.0e300)) *flag = 1;
                rv[c] = pivot_rcp(piv);
            }
        }
        if (idl) {
#pragma unroll
            for (int k = 0; k < 16; ++k) Xm[(base + k) * DL + base + lane] = a[k];
        }
    };
    // G_bb = (Un_bb^T)^-1 (unit lower) by forward substitution: lane c (mod 16) solves
    // Un_bb^T x = e_c; entry [i][m] of Un_bb^T is Un[m][i], a wavefront-uniform LDS read
    auto tinv = [&](int b) {
        const int base = 16 * b, c = here(fr);
        double sv[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) sv[i] = (i == c) ? 1.0 : 0.0;
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const double xm = sv[m] * rv[base + m];
#pragma unroll
            for (int i = m + 1; i < 16; ++i) sv[i] -= Am[(base + m) * DL + base + i] * xm;
        }
        if (lane < 16) {
#pragma unroll
            for (int i = 0; i < 16; ++i) Xm[(base + i) * DL + base + c] = sv[i];
        }
        __builtin_amdgcn_wave_barrier();
    };
    // trailing tiles: A_ij -= Un_bi^T U_bj for b < i <= j
    auto trail = [&](int b) {
        const int base = 16 * b;
        int t = 0;
        for (int i = b + 1; i < 4; ++i)
            for (int j = i; j < 4; ++j, ++t) {
                if ((t & (NT / 64 - 1)) != wave) continue;
                d4 acc;
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[v] = Am[(16 * i + 4 * v + fq) * DL + 16 * j + fr];
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    acc = mfma4(-Am[(base + 4 * ks + fq) * DL + 16 * i + fr] * rv[base + 4 * ks + fq],
                                Am[(base + 4 * ks + fq) * DL + 16 * j + fr], acc);
#pragma unroll
                for (int v = 0; v < 4; ++v) Am[(16 * i + 4 * v + fq) * DL + 16 * j + fr] = acc[v];
            }
    };
    // G = (Un11^T)^-1: tile T_im of Un11^T is Un_mi transposed
    block_schedule(Xm, sweep, tinv, trail, [&](int i, int m, int ks) {
        return Am[(16 * m + 4 * ks + fq) * DL + 16 * i + fr] * rv[16 * m + 4 * ks + fq]; }, beside, ahead);
}

// t = big (big + 1) / 2 + small, 0 <= small <= big
__device__ __forceinline__ void tri_decode(int t, int& big, int& small)
{
    int i = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
    while ((i + 1) * (i + 2) / 2 <= t) ++i;
    while (i * (i + 1) / 2 > t) --i;
    big = i;
    small = t - i * (i + 1) / 2;
}

}  // namespace fobq
