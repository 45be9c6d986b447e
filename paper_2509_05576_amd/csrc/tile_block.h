// 64 x 64 diagonal blocks of the factorizations, held in LDS by one workgroup (device code shared by factor.hip and
// flow.hip).
#pragma once
#include <type_traits>

#include "fobq_internal.h"

namespace fobq {

constexpr int NB = 64;

// ---------------------------------------------------------------------------
// 64 x 64 diagonal blocks.  Both diagonal-block kernels keep the block in LDS and
// work on it as a 4 x 4 grid of 16 x 16 tiles.  The only sequential arithmetic is
// the unblocked sweep over the 16 pivots of a diagonal tile: one wavefront, one
// row (Cholesky) or column (elimination) of the whole block per lane, so the same
// sweep also produces the tiles below (right of) the diagonal tile, and, in lanes it
// would leave idle, the triangular inverse of the diagonal tile.  A wavefront on its
// own issues one instruction of any kind per 5 to 8 cycles, and a value that goes
// through v_readlane or LDS to other lanes is late by as much again; so every row of 16
// lanes keeps a copy of the diagonal tile, and pivots and multipliers reach the lanes as
// DPP operands of the multiply-adds themselves.  Everything else --
// trailing update, assembly of the 64 x 64 triangular inverse from the tile
// inverses -- is 16 x 16 x 16 products on the matrix cores (4 MFMAs each), one tile
// per wavefront, one interval behind the sweeps.
typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int NT = 512;   // threads per workgroup of every kernel that uses these routines (8 wavefronts)
constexpr int DL = 66;    // LDS row stride (doubles): conflict-free 8-byte MFMA fragment reads per half-wave
constexpr int SWEEP_LDS = NB + 16 * DL + 2;   // doubles of LDS that chol_block / elim_block need besides the two tiles

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

// Lane K of every row of 16 lanes, to the whole row (DPP row_newbcast, which 64-bit operations take).  The compiler does not see
// into the asm and so does not keep the two wait states that DPP wants between a vector instruction and the one that reads its
// result across lanes: every statement brings its own where the value may be that young, and row_factor hands on a factor
// that is old enough for any number of uses.  That nothing lands in between (a copy, a spill) the build checks in its listing.
template <int K>
__device__ __forceinline__ double row_lane(double v)
{
    double x;
    asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%c2 row_mask:0xf bank_mask:0xf" : "=v"(x) : "v"(v), "n"(K));
    return x;
}
__device__ __forceinline__ double row_factor(double a, double b)      // a * b
{
    double x;
    asm("v_mul_f64 %0, %1, %2\n\ts_nop 1" : "=v"(x) : "v"(a), "v"(b));
    return x;
}
// acc -= (lane K of f) * m
template <int K>
__device__ __forceinline__ void row_update(double& acc, double f, double m)
{
    asm("v_fmac_f64_dpp %0, -%1, %2 row_newbcast:%c3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(f), "v"(m), "n"(K));
}
template <int K, int N, class F>
__device__ __forceinline__ void unroll(F f)           // f(integral_constant<K>) .. f(integral_constant<N - 1>)
{
    if constexpr (K < N) {
        f(std::integral_constant<int, K>{});
        unroll<K + 1, N>(f);
    }
}

__device__ __forceinline__ void identity_rows(double* idt, int fr, int fq)
{
#pragma unroll
    for (int u = 0; u < 4; ++u) idt[(4 * u + fq) * DL + fr] = 4 * u + fq == fr ? 1.0 : 0.0;
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

// Schedule shared by chol_block and elim_block.  sweep(b): pivots of diagonal tile b, the
// tiles below / right of it and the inverse X_bb of the diagonal tile; trail(b): update of the tiles
// behind tile row/column b; tf: tile fetch for inv_tile.
//   interval   wavefront 0        wavefront 1   wavefront 2   wavefronts 3, 4, 5
//   b = 0      sweep(0)
//   b = 1      sweep(1)
//   b = 2      sweep(2)                         X_10
//   b = 3      sweep(3)           X_21          X_20          the sums of X_30, X_31, X_32 as far as they
//                                                             do not need this interval's tiles
//   then                                                      rest of the sums, times -X_33
//   (after each of b = 0..2: trail(b) on all wavefronts)
// Called by all NT threads of the workgroup (at least 6 wavefronts); ends with a barrier.
// `beside` is called by wavefronts 1 .. 7 during the first sweep: the caller's work on tiles of the block that this sweep does
// not read (it reads the first tile column / row only).  `ahead` is called by every wavefront about 2 us before the end (wavefront 0: after the last sweep).
struct Nothing { __device__ void operator()() const {} };
template <class SW, class TR, class TF, class BS, class AH>
__device__ __forceinline__ void block_schedule(double* Xm, SW sweep, TR trail, TF tf, BS beside, AH ahead)
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
//        Xm = L^-1 (lower);  scratch: SWEEP_LDS doubles of LDS
//   flag: set to 1 when a pivot is <= 0 or not finite (the pivot is replaced by 1 so that
//         the arithmetic stays finite; the caller reports ENOTPD).
// Called by all NT threads of the workgroup; ends with a barrier.
template <class BS = Nothing, class AH = Nothing>
__device__ __forceinline__ void chol_block(double* Am, double* Xm, double* scratch, int* __restrict__ flag, BS beside = BS(), AH ahead = AH())
{
    const int tid = here(threadIdx.x), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 15, fq = lane >> 4;
    double* idt = scratch;     // 16 rows of the identity, row stride DL: written and read by the wavefront of the sweeps
    if (wave == 0) identity_rows(idt, fr, fq);

    // Right-looking Cholesky of the 16 columns base .. base+15 of the block over all rows >= base.  Every row of 16
    // lanes holds the diagonal tile (lane s tile row s; what lies right of its diagonal is carried along and never
    // used), so the pivot and the multipliers of the columns are operands of the instructions that use them, and beside
    // it, lane rho, row rho of the block below the tile (their part of L: l_rho,k = (a_rho,k - sum l l) / l_kk), or,
    // in the lanes of the tile itself, the rows of the identity, which become I L_bb^-T: lane s ends with column s of
    // X_bb = L_bb^-1.  The lanes above idle on rows of the identity.
    auto sweep = [&](int b) {
        const int base = 16 * b, own = lane >> 4;
        const double* tile = Am + (base + fr) * DL + base;
        const double* src = own > b ? Am + lane * DL + base : idt + fr * DL;
        double t[16], a[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) t[j] = tile[j];
#pragma unroll
        for (int j = 0; j < 16; ++j) a[j] = src[j];
        // The chain per pivot: broadcast, reciprocal square root, multiply, multiply-add.  Beside it the updates by
        // the pivot before of the columns that are not next.
        double tp = 0.0;
        unroll<0, 16>([&](auto K) {
            constexpr int k = K;
            const double rs = pivot_rsqrt(row_lane<k>(t[k]));              // 1 / L[k][k]
            if constexpr (k > 0) {
                row_update<k>(a[k], tp, a[k - 1]);
                unroll<k + 1, 16>([&](auto J) {
                    row_update<J>(t[J], tp, t[k - 1]);
                    row_update<J>(a[J], tp, a[k - 1]);
                });
            }
            t[k] = row_factor(t[k], rs);                                   // l_sk (a pivot's own lane: sqrt)
            a[k] *= rs;
            if constexpr (k < 15) row_update<k + 1>(t[k + 1], t[k], t[k]);
            tp = t[k];
        });
        if (own > b) {
#pragma unroll
            for (int j = 0; j < 16; ++j) Am[lane * DL + base + j] = a[j];
        } else if (own == b) {
#pragma unroll
            for (int j = 0; j < 16; ++j) Am[lane * DL + base + j] = t[j];
#pragma unroll
            for (int k = 0; k < 16; ++k) Xm[(base + k) * DL + lane] = a[k];
            // A pivot that is not a positive normal number (nor anything after it) leaves no positive
            // finite L[r][r] behind: one test per tile row after the sweep instead of one per pivot.
            const double lrr = Am[lane * DL + lane];
            if (!(lrr > 0.0) || !(lrr < 1.0e300)) *flag = 1;
        }
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
    block_schedule(Xm, sweep, trail,
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
    double* idt = rv + NB;     // as in chol_block
    if (wave == 0) identity_rows(idt, fr, fq);

    // Elimination of the 16 pivots base .. base+15 over all columns >= base, laid out as in chol_block by columns: every row
    // of 16 lanes holds the diagonal tile (lane s tile column s; what lies below its diagonal is carried along and
    // never used), beside it lane c column c of the pivot rows right of the tile, or in the lanes of the tile
    // itself the columns of the identity, which become G_bb I: lane s ends with column s of G_bb = (Un_bb^T)^-1.
    auto sweep = [&](int b) {
        const int base = 16 * b, own = lane >> 4;
        const double* tile = Am + base * DL + base + fr;
        const double* src = own > b ? Am + base * DL + lane : idt + fr;
        double t[16], a[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) t[j] = tile[j * DL];
#pragma unroll
        for (int j = 0; j < 16; ++j) a[j] = src[j * DL];
        double tp = 0.0, ap = 0.0;                                         // Un of the pivot row before
        unroll<0, 16>([&](auto K) {
            constexpr int k = K;
            const double pi = pivot_rcp(row_lane<k>(t[k]));
            if constexpr (k > 0) {
                row_update<k>(a[k], t[k - 1], ap);
                unroll<k + 1, 16>([&](auto J) {
                    row_update<J>(t[J], t[k - 1], tp);
                    row_update<J>(a[J], t[k - 1], ap);
                });
            }
            tp = t[k] * pi;                                                // Un[k][s]; t[k] = U[k][s]
            ap = a[k] * pi;
            if constexpr (k < 15) row_update<k + 1>(t[k + 1], t[k], tp);
        });
        if (own > b) {
#pragma unroll
            for (int k = 0; k < 16; ++k) Am[(base + k) * DL + lane] = a[k];
        } else if (own == b) {
#pragma unroll
            for (int k = 0; k < 16; ++k) Am[(base + k) * DL + lane] = t[k];   // U[k][c] for k <= c
#pragma unroll
            for (int k = 0; k < 16; ++k) Xm[(base + k) * DL + lane] = a[k];
            // a pivot that is not a positive normal number leaves such a value, or a NaN, on the diagonal
            const double piv = Am[lane * DL + lane];
            if (!(piv > 0.0) || !(piv < 1.0e300)) *flag = 1;
            rv[lane] = pivot_rcp(piv);
        }
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
    block_schedule(Xm, sweep, trail, [&](int i, int m, int ks) {
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
