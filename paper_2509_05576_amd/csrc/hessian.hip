// Hessian of the layer objective (Section 3, Eq. 2): H = (2/N) X X^T.
//
// xxt_kernel: fp32 X is read from HBM, staged through LDS as fp32, widened to
// fp64 when the MFMA fragments are formed (products of two fp32 values are
// exact in fp64), and accumulated with v_mfma_f64_16x16x4_f64.  Only the tiles (128 or 64 wide;
// in long calls 160 for 129 to 160 columns and 96 for 257 to 288, see xxt_tile) on or below the diagonal are
// computed, and of a diagonal tile only the 16 x 16 MFMA tiles on or below its diagonal (36 of 64;
// not at 64, see xxt_diag_cost).
//
// Work decomposition ("stream-K"): the work items are (tile, 32-column chunk of
// the calibration dimension) pairs in tile-major order, diagonal tiles first; a
// fixed number of persistent workgroups each take one contiguous range of items,
// all ranges equally expensive (an item of a diagonal tile is priced below one of
// another tile), so every workgroup does the same amount of work whatever d and n are.  A
// range can cross tile boundaries; the part of a tile done by one workgroup is a
// "piece".  Piece p of a tile is added into slab p of Hpart (d x d each; the first
// launch of an accumulation stores it there), and exactly one workgroup owns a given (tile, piece) in a launch, so
// the sums do not depend on the order in which workgroups finish.
//
// Convolution mode: the same kernel with a loader that reads the unfolded input of a k x k
// convolution straight from NHWC feature maps (X is never materialised).  Row (c, ky, kx) of
// X, column (image, y, x) is maps[image][y*stride + ky - pad][x*stride + kx - pad][c] or 0
// outside the map.  pad_maps_kernel first writes a zero-padded copy of the maps with one extra
// all-zero image at the end, so that every window lies inside the copy (no per-element test)
// and the columns past the last pixel read zeros from the extra image (no branch).  Inside the
// kernel the rows are taken tap-major (row' = (ky*k + kx)*C + c) so that consecutive rows are
// consecutive channels, which NHWC stores contiguously; the finalize kernel of this mode puts
// H back into the (c, ky, kx) order.
#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

#include "fobq_internal.h"

namespace fobq {

typedef double d4 __attribute__((ext_vector_type(4)));

// n / dv for 0 <= n < 2^32 and a divisor fixed at launch: q = (t + ((n - t) >> s1)) >> s2 with
// t = umulhi(m, n)  (division by an invariant integer through multiplication).
struct FastDiv { uint32_t m; int s1, s2; };

static FastDiv fastdiv_make(uint32_t dv)
{
    FastDiv f;
    int L = 0;
    while ((1ull << L) < dv) ++L;
    f.m = (uint32_t)(((1ull << 32) * ((1ull << L) - dv)) / dv + 1);
    f.s1 = L < 1 ? L : 1;
    f.s2 = L > 1 ? L - 1 : 0;
    return f;
}

__device__ __forceinline__ uint32_t fastdiv(uint32_t n, const FastDiv& f)
{
    const uint32_t t = __umulhi(f.m, n);
    return (t + ((n - t) >> f.s1)) >> f.s2;
}

struct ConvP {
    int hp, wp, c, k, stride, ho, wo;   // hp, wp: height and width of the padded copy
    int64_t zero_origin;                // element offset of the all-zero image
    FastDiv div_img;    // by ho * wo
    FastDiv div_row;    // by wo
    FastDiv div_c;      // by c
    FastDiv div_k;      // by k
};

// out: (n_img + 1) x hp x wp x c, hp = h + 2 pad, wp = w + 2 pad; image n_img is all zeros.  Bound by memory: a workgroup takes
// rows of the padded copy (zeros, the row of the map, zeros: no division per element) or (SPLIT), where the rows are few and long,
// one of `parts` runs of `run` pixels of a row; 16 bytes per lane where the channels come in fours (VEC: c % 4 == 0, both pointers
// 16-byte aligned).  AMAX: the maxima |.| of every channel (bit patterns) are taken on the way: the first `active` threads walk a
// run in steps of a multiple of c, so that a thread stays on its channels; one atomic per channel and workgroup.  The 64-image
// 56 x 56 x 128 maps (103 MB): 85 us for a copy by elements and 139 us for a second pass over it with an atomic per thread, 42 us
// together now.  One image of 1 x 100352 x 256 (two rows of 103 MB; the whole accumulate call, 1 x 1): 3.56 ms with undivided
// rows, 0.36 with the copy by elements, 0.23 in runs.
template <bool VEC, bool AMAX, bool SPLIT>
__global__ __launch_bounds__(256) void pad_maps_kernel(const float* __restrict__ maps, int n_img, int h, int w, int c, int pad,
                                                       float* __restrict__ out, int64_t rows, int parts, int run, int active,
                                                       unsigned* __restrict__ amax)
{
    typedef typename std::conditional<VEC, float4, float>::type V;
    constexpr int VL = VEC ? 4 : 1;
    const int hp = h + 2 * pad;
    const int unit = c / VL, lead = pad * unit, len = w * unit, total = len + 2 * lead;
    V zero{};
    unsigned m[VL];
#pragma unroll
    for (int e = 0; e < VL; ++e) m[e] = 0;
    const int64_t items = SPLIT ? rows * parts : rows;
    for (int64_t item = blockIdx.x; item < items; item += gridDim.x) {
        const int64_t row = SPLIT ? (int)item / parts : item;       // (SPLIT: at most 2048 items)
        const int part = SPLIT ? (int)item - (int)row * parts : 0;
        const bool first = !SPLIT || part == 0, last = !SPLIT || part == parts - 1;
        const int64_t img = row / hp;
        const int y = (int)(row - img * hp) - pad;
        V* __restrict__ dst = reinterpret_cast<V*>(out) + row * total;
        if (img >= n_img || (unsigned)y >= (unsigned)h) {
            const int end = last ? total : (part + 1) * run * unit;
            for (int x = part * run * unit + threadIdx.x; x < end; x += 256) dst[x] = zero;
            continue;
        }
        const V* __restrict__ src = reinterpret_cast<const V*>(maps) + (img * h + y) * len;
        if (first || last)
            for (int x = threadIdx.x; x < lead; x += 256) {
                if (first) dst[x] = zero;
                if (last) dst[lead + len + x] = zero;
            }
        if ((int)threadIdx.x < active) {
            const int end = last ? len : (part + 1) * run * unit;
#pragma unroll 4
            for (int x = part * run * unit + threadIdx.x; x < end; x += active) {
                const V v = src[x];
                if (AMAX) {
                    const float* f = reinterpret_cast<const float*>(&v);
#pragma unroll
                    for (int e = 0; e < VL; ++e) m[e] = max(m[e], __float_as_uint(f[e]) & 0x7fffffffu);
                }
                dst[lead + x] = v;
            }
        }
    }
    if (AMAX) {
        __shared__ unsigned part[256 * VL];
#pragma unroll
        for (int e = 0; e < VL; ++e) part[threadIdx.x * VL + e] = m[e];      // thread t: channels (t VL + e) % c
        __syncthreads();
        for (int ch = threadIdx.x; ch < c; ch += 256) {
            unsigned best = 0;
            for (int i = ch; i < active * VL; i += c) best = max(best, part[i]);
            atomicMax(&amax[ch], best);
        }
    }
}

// aligned: both pointers to 16 bytes
PadPlan pad_maps_plan(int64_t n_img, int h, int w, int c, int pad, bool aligned, bool maxima)
{
    PadPlan p;
    p.rows = (n_img + 1) * (h + 2 * pad);
    p.vec = aligned && c % 4 == 0;
    const int unit = p.vec ? c / 4 : c;                // steps of a row after which the channels repeat
    p.maxima = maxima && unit <= 256;
    p.active = p.maxima ? unit * (256 / unit) : 256;
    // the maxima cost an atomic per channel and workgroup: 2048 workgroups 61 us, 768 42 us (64 x 56 x 56 x 128; 128 x 14 x 14 x
    // 256: 43 and 23)
    const int64_t most = p.maxima ? 768 : 2048;
    // fewer rows than that: cut into parts of at least four steps of a whole workgroup
    const int64_t fill = most / p.rows, steps = (int64_t)w * unit / (4 * 256);
    p.parts = (int)std::max<int64_t>(1, std::min(std::min(fill, steps), (int64_t)w));
    p.run = (w + p.parts - 1) / p.parts;
    p.parts = (w + p.run - 1) / p.run;                // none of them empty
    p.wgs = (int)std::min(p.rows * p.parts, most);
    return p;
}

// amax: null, or c words that hold zeros; *took (if amax): whether the maxima were taken (else the caller's own pass does it)
hipError_t launch_pad_maps(hipStream_t s, const float* maps, int n_img, int h, int w, int c, int pad, float* out, unsigned* amax, bool* took,
                           hipEvent_t done)
{
    const PadPlan p = pad_maps_plan(n_img, h, w, c, pad, ((reinterpret_cast<uintptr_t>(maps) | reinterpret_cast<uintptr_t>(out)) & 15) == 0, amax != nullptr);
    if (took) *took = p.maxima;
    auto launch = [&](auto whole, auto split) {
        hipExtLaunchKernelGGL((p.parts > 1 ? split : whole), dim3(p.wgs), dim3(256), 0, s, nullptr, done, 0, maps, n_img, h, w, c, pad, out, p.rows,
                              p.parts, p.run, p.active, amax);
    };
    if (p.vec && p.maxima) launch(pad_maps_kernel<true, true, false>, pad_maps_kernel<true, true, true>);
    else if (p.vec)        launch(pad_maps_kernel<true, false, false>, pad_maps_kernel<true, false, true>);
    else if (p.maxima)     launch(pad_maps_kernel<false, true, false>, pad_maps_kernel<false, true, true>);
    else                   launch(pad_maps_kernel<false, false, false>, pad_maps_kernel<false, false, true>);
    return hipGetLastError();
}

// Tile edge XT: 128 (each of the 4 wavefronts owns 64 x 64 = 4 x 4 MFMA tiles); 96 (48 x 48 = 3 x 3) or 64 (32 x 32 =
// 2 x 2; twice the operand traffic and conversions per MFMA) where 128-wide tiles are mostly padding; 160 for a d that a
// single tile holds, which is a diagonal one: 8 wavefronts share the 55 MFMA tiles of its lower triangle and X is read once.
constexpr int XK = 32;           // calibration columns per LDS stage
constexpr int XLD = XK + 4;      // fp32 row stride in LDS: 16B-aligned rows, conflict-free 16B fragment reads
constexpr int xxt_waves(int xt) { return xt == 160 ? 8 : 4; }
constexpr int xxt_wgs(int xt) { return xt == 64 ? 1024 : xt == 160 ? 256 : 512; }   // persistent workgroups: 4, 1 or 2 per compute unit

// Price of one chunk of a diagonal tile in units of 1/16 of another tile's chunk.  A 128 x 128 diagonal tile
// is 8 x 8 MFMA tiles of which the 36 on and below its diagonal are needed: 9 per wavefront (diag_mma), and one
// operand panel instead of two.  By MFMA count that is 9/16; the loads, LDS stores and barriers per chunk stay,
// and the ranges come out equally long in time at 10/16 (plain loader) and 12/16 (convolution loader: more
// address arithmetic per chunk) -- measured: with 9 the workgroups on the diagonal tiles finish last.  A 96 x 96
// diagonal tile has 6 per wavefront of the 9 of a full one.
// A 64 x 64 tile has 4 x 4 MFMA tiles, 10 needed: no split over 4 wavefronts beats the 4 each of the full tile.
constexpr int xxt_diag_cost(int xt, bool conv) { return xt == 128 ? (conv ? 12 : 10) : xt == 96 ? (conv ? 13 : 12) : 16; }
constexpr int xxt_diag_cost_min(int xt) { return xxt_diag_cost(xt, false); }

// Tile edge for d columns: 128, or 64 where that spends less than 5/6 of the MFMA tiles ...
static int xxt_base_tile(int d)
{
    const int64_t n128 = (d + 127) / 128, n64 = (d + 63) / 64;
    const int64_t a128 = n128 * (n128 + 1) / 2 * 128 * 128, a64 = n64 * (n64 + 1) / 2 * 64 * 64;
    return a64 * 6 < a128 * 5 ? 64 : 128;
}

// ... and in long calls 160 or 96, by the MFMA tiles per chunk that each choice spends (a diagonal tile by its price), over the
// part of the matrix rate that it reaches there (measured at d = 128, 147, 288, 1024): 64: 0.73, 96: 0.66, 128: 0.92, 160: 0.60;
// 5 % in favour of the choice above.  That comes to 160 for 129 to 160 columns and 96 for 257 to 288.
static int xxt_long_tile(int d)
{
    auto cost = [&](int xt) {
        const int64_t n = (d + xt - 1) / xt, mt = xt / 16, full = mt * mt;
        return xt == 160 ? (n == 1 ? 56.0 : 1e30) : (double)(n * full * xxt_diag_cost(xt, true) / 16 + n * (n - 1) / 2 * full);
    };
    const int base = xxt_base_tile(d);
    if (d <= 128) return base;               // few products: a tile is cut into so many pieces that their sums weigh more
    const double own = cost(base) / (base == 64 ? 0.73 : 0.92);
    if (cost(160) / 0.60 < own) return 160;
    return cost(96) / 0.66 < 0.95 * own ? 96 : base;
}

// A short call is over before the wide tiles' matrix rate counts, and their longer prologue and epilogue, on fewer workgroups, remain.
// Accumulate calls after the first, 64 wide and wide: 147 columns of X, n = 256 6.9 and 12.7 us, 2048 12.8 and 17.5, 4096 23.2 and
// 23.3, 6144 35.6 and 30.0, 65536 76 and 65; 288 columns, n = 256 7.1 and 11.7, 8192 33.5 and 39.6, 16384 49.7 and 48.7, 24576
// 64.2 and 60.1, from 32-channel maps 16384 56.8 and 60.6, 25600 74.4 and 74.6, 51200 126 and 113, 400000 826 and 685.
int xxt_tile(int d, int64_t n)
{
    const int wide = xxt_long_tile(d);
    return n < (wide == 160 ? 4096 : wide == 96 ? 24576 : 0) ? xxt_base_tile(d) : wide;
}

// The MFMA tiles on and below the diagonal of a B x B grid in the order in which they are dealt to the wavefronts, K
// consecutive ones each: rows 0, B - 1, 1, B - 2, ...  (B = 8, K = 9: rows w and 7 - w for wavefront w).
template <int B>
struct TriOrder {
    signed char r[B * (B + 1) / 2], c[B * (B + 1) / 2];
    constexpr TriOrder() : r(), c()
    {
        int t = 0;
        for (int x = 0; x < B; ++x) {
            const int row = x % 2 == 0 ? x / 2 : B - 1 - x / 2;
            for (int col = 0; col <= row; ++col, ++t) { r[t] = (signed char)row; c[t] = (signed char)col; }
        }
    }
    constexpr bool needs(int t0, int t1, int row) const      // fragment `row` is an operand of the tiles t0 .. t1 - 1
    {
        for (int t = t0; t < t1 && t < B * (B + 1) / 2; ++t)
            if (r[t] == row || c[t] == row) return true;
        return false;
    }
};

// the place of tile t in that order (two consecutive rows from an even x on have B + 1 tiles, the first of them x / 2 + 1)
template <int B>
__device__ __forceinline__ bool tri_place(int t, int& r, int& c)
{
    const int pair = t / (B + 1), u = t - pair * (B + 1);
    const bool second = u > pair;
    r = second ? B - 1 - pair : pair;
    c = second ? u - pair - 1 : u;
    return t < B * (B + 1) / 2;
}

// One group of 16 calibration columns of a diagonal tile for wavefront W: its K MFMA tiles in TriOrder's order.  Both
// operands come from the one panel At.
template <int W, int B, int K, class F>
__device__ __forceinline__ void diag_mma(const float (*At)[XLD], int g, int fr, int fk, d4 (&acc)[K], F after_step)
{
    constexpr TriOrder<B> o;
    constexpr int T0 = W * K, T1 = T0 + K < B * (B + 1) / 2 ? T0 + K : B * (B + 1) / 2;
    float4 f[B];
#pragma unroll
    for (int j = 0; j < B; ++j)
        if (o.needs(T0, T1, j)) f[j] = *reinterpret_cast<const float4*>(&At[j * 16 + fr][g * 16 + fk]);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        double b[B];
#pragma unroll
        for (int j = 0; j < B; ++j)
            if (o.needs(T0, T1, j)) b[j] = (double)(ks == 0 ? f[j].x : ks == 1 ? f[j].y : ks == 2 ? f[j].z : f[j].w);
#pragma unroll
        for (int t = T0; t < T1; ++t) acc[t - T0] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[o.r[t]], b[o.c[t]], acc[t - T0], 0, 0, 0);
        after_step(ks);     // the convolution loader's share of this k-step
    }
}

// Order of the tiles.  The nt diagonal tiles come first, in order; the tiles below the diagonal follow as the
// lower triangle (with its diagonal) of an (nt - 1) x (nt - 1) grid whose row r stands for tile row r + 1, in
// this order of such a triangle: tile rows are taken in pairs (2r, 2r + 1) and a pair is walked
// column by column, (2r, J), (2r + 1, J), (2r, J + 1), ...  Consecutive tiles of the order then share a
// panel of X: the column panel J with the tile just before or after, the row panel with the tile two
// places away.  Pair r starts at index 2 r^2 + r and has 4 r + 3 tiles; an odd last row stands alone.
__device__ __forceinline__ void tile_decode(int t, int nt, int& I, int& J)
{
    int r = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.25f);
    while (2 * (r + 1) * (r + 1) + (r + 1) <= t) ++r;
    while (2 * r * r + r > t) --r;
    const int u = t - (2 * r * r + r);
    if (2 * r + 1 >= nt) { I = 2 * r; J = u; }                       // unpaired last row
    else if (u < 4 * r + 2) { I = 2 * r + (u & 1); J = u >> 1; }
    else { I = 2 * r + 1; J = 2 * r + 1; }                           // diagonal tile of the second row
}

// MODE 0: X rows are 16-byte aligned (ld % 4 == 0, base aligned) -> float4 loads.
// MODE 1: any ld / alignment.  MODE 2: X = feature maps, n = images * ho * wo (convolution mode).
template <int MODE, int XT>
__global__ __launch_bounds__(64 * xxt_waves(XT), XT == 64 ? 4 : 2) void xxt_kernel(const float* __restrict__ X, int64_t ld, int d, int64_t n,
                                                     double* __restrict__ Hpart, int chunks, int64_t range_cost,
                                                     int64_t total_items, int classes, int splits, int fresh, ConvP cp)
{
    constexpr bool FAST = MODE == 0;
    constexpr bool CONV = MODE == 2;
    constexpr int NW = xxt_waves(XT);
    constexpr int RW = 8 * NW;        // rows per group of the plain loader (one float4 per row and 8 threads)
    constexpr int RG = (XT + RW - 1) / RW;
    constexpr int PX = XK / NW;       // pixels per wavefront and chunk (convolution loader)
    constexpr bool SINGLE = XT == 160;   // the one tile is a diagonal one
    constexpr bool LOWER = XT != 64;  // of a diagonal tile only the lower triangle is formed, from one panel
    constexpr int WT = XT / 2;        // edge of a wavefront's part of the tile
    constexpr int MT = SINGLE ? 1 : WT / 16;       // MFMA tiles per edge of that part
    constexpr int TB = XT / 16, TK = (TB * (TB + 1) / 2 + NW - 1) / NW;   // diagonal tile: MFMA tiles per edge, per wavefront
    __shared__ float As[2][XT][XLD];
    __shared__ float Bs[2][SINGLE ? 1 : XT][XLD];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int lr = tid >> 3;          // row within a group of RW rows
    const int lk = (tid & 7) * 4;     // 0..28: first of 4 consecutive calibration columns
    const int fr = lane & 15;         // fragment row
    const int fk = (lane >> 4) * 4;   // fragment: 4 consecutive columns, one per k-step (the sum over k is order-free)
    const int wave_s = __builtin_amdgcn_readfirstlane(wave);   // the same value, known to be wavefront-uniform

    // Workgroups are dealt to the 8 XCDs round-robin; give each XCD one contiguous run of ranges, so
    // that the workgroups sharing an L2 work on neighbouring tiles (which share panels of X) at almost
    // the same position of the calibration dimension.
    const int nx = 8, gq = (int)gridDim.x / nx, grem = (int)gridDim.x % nx;
    const int xcd = (int)blockIdx.x % nx;
    const int vpos = xcd * gq + min(xcd, grem) + (int)blockIdx.x / nx;
    // Position vpos in that XCD-contiguous order -> range index vb, class-major: when a tile is cut
    // into `classes` pieces, the ranges vb = c, c + classes, c + 2 classes, ... cover the same part
    // of the calibration dimension of consecutive tiles, and only they can share fetches; ordering
    // the ranges by (vb mod classes, vb) puts up to 64 of them on one XCD instead of 64 / classes.
    int vb = vpos;
    if (classes > 1) {
        int cls = 0, before = 0;
        for (;;) {
            const int cnt = ((int)gridDim.x - cls + classes - 1) / classes;   // ranges with vb mod classes == cls
            if (vpos < before + cnt) break;
            before += cnt;
            ++cls;
        }
        vb = cls + classes * (vpos - before);
    }
    const int nt = (d + XT - 1) / XT;

    // This workgroup's range of items [g0, g1) and its pieces (one per tile it touches).  All
    // workgroups start together and advance one chunk per step, so chunk k is best visited at step
    // k mod per_wg: workgroups on neighbouring tiles (which share panels of X and, thanks to the
    // mapping above, an L2) then read the same columns of X at the same time.  A range inside one
    // tile therefore starts at its chunk whose index is a multiple of per_wg and wraps around; a range
    // over two tiles takes the head of the later tile (chunks 0 ...) before the tail of the earlier
    // one.  The order of the sum over chunks is free; it stays fixed, so results are reproducible.
    // Items are laid out with the nt diagonal tiles first, then the tiles below the diagonal.  A chunk of
    // a diagonal tile costs WD units of work (see xxt_diag_cost), any other 16; the
    // ranges are equally long in cost, and both ends of a range are rounded down to an item in the same way.
    constexpr int WD = xxt_diag_cost(XT, CONV);
    const int64_t diag_items = (int64_t)nt * chunks, diag_cost = diag_items * WD;
    auto item_at = [&](int64_t x) { return x < diag_cost ? x / WD : diag_items + (x - diag_cost) / 16; };
    const int64_t g0 = min(total_items, item_at((int64_t)vb * range_cost));
    const int64_t g1 = min(total_items, item_at((int64_t)(vb + 1) * range_cost));
    if (g0 >= g1) return;
    const int t_first = (int)(g0 / chunks), t_last = (int)((g1 - 1) / chunks);
    const int npieces = t_last - t_first + 1;

    for (int pi = 0; pi < npieces; ++pi) {
        const int tile = npieces == 2 ? t_last - pi : t_first + pi;
        const int64_t tile_first = (int64_t)tile * chunks;
        const int c_begin = (int)(max(g0, tile_first) - tile_first);
        const int c_end = (int)(min(g1, tile_first + chunks) - tile_first);
        const int len = c_end - c_begin;
        const bool diag = tile < nt;
        const int64_t per_wg = max((int64_t)1, range_cost / (diag ? WD : 16));   // nominal range length in this tile's chunks
        const bool load_b = !SINGLE && !(LOWER && diag);     // a diagonal tile's two operand panels are one: only As is filled
        int rot = 0;
        if (npieces == 1) {
            const int64_t aligned = (c_begin + per_wg - 1) / per_wg * per_wg;
            if (aligned < c_end) rot = (int)(aligned - c_begin);
        }
        auto chunk_at = [&](int i) {
            int c = i + rot;
            if (c >= len) c -= len;
            return c_begin + c;
        };
        // piece index of this range inside its tile: number of workgroup boundaries before it
        // 0 for the workgroup whose range reaches the tile first
        int64_t first_range = (diag ? tile_first * WD : diag_cost + (tile_first - diag_items) * 16) / range_cost;
        while (first_range < vb && item_at((first_range + 1) * range_cost) <= tile_first) ++first_range;
        const int piece = min((int)(vb - first_range), splits - 1);   // (the host sizes the ranges so that it is < splits)
        int I, J;
        if (diag) { I = tile; J = tile; }
        else { tile_decode(tile - nt, nt - 1, I, J); ++I; }
        const int i0 = I * XT, j0 = J * XT;

        // plain modes: clamped row pointers (rows past d produce outputs that are never stored);
        // thread = (row lr + RW u, 4 consecutive columns)
        const float* __restrict__ arow[RG];
        const float* __restrict__ brow[RG];
        // convolution mode: thread = (rows lane + 64 q, pixels PX wave + j): a load covers 64
        // consecutive channels (256 contiguous bytes) of ONE pixel, so the pixel's decoding and its
        // window origin are wavefront-uniform (scalar unit).  Per tile: the offset of this thread's
        // two rows (ky, kx, channel) of each operand from the window's top-left element in the
        // padded copy.  Rows past d stand in as row d - 1.
        constexpr int QN = (XT + 63) / 64;    // rows per operand and thread in convolution mode (those past the tile are not stored)
        uint32_t offA[QN], offB[QN];
        if (CONV) {
#pragma unroll
            for (int q = 0; q < QN; ++q) {
                const int ra = min(i0 + lane + 64 * q, d - 1), rb = min(j0 + lane + 64 * q, d - 1);
                const uint32_t ta = fastdiv((uint32_t)ra, cp.div_c), tb = fastdiv((uint32_t)rb, cp.div_c);
                const uint32_t kya = fastdiv(ta, cp.div_k), kyb = fastdiv(tb, cp.div_k);
                offA[q] = (kya * cp.wp + (ta - kya * cp.k)) * cp.c + ((uint32_t)ra - ta * cp.c);
                offB[q] = (kyb * cp.wp + (tb - kyb * cp.k)) * cp.c + ((uint32_t)rb - tb * cp.c);
            }
        } else {
#pragma unroll
            for (int u = 0; u < RG; ++u) {
                arow[u] = X + (int64_t)min(i0 + lr + RW * u, d - 1) * ld;
                brow[u] = X + (int64_t)min(j0 + lr + RW * u, d - 1) * ld;
            }
        }
        constexpr int PN = CONV ? QN * PX / 4 : RG;
        float4 pa[PN], pb[PN];
        // Convolution mode: the loads of pixel j (0..PX-1) of chunk c for this thread's rows; called
        // with j = 0, 1, ..., PX - 1 in this order.  Pixel 0 is decoded in full (two divisions by
        // invariant integers), the others by stepping (image, y, x) one pixel on; a pixel past the
        // last one takes the all-zero image.  All of it is wavefront-uniform, i.e. scalar-unit
        // work with no branch: arithmetic on the vector unit takes cycles from the fp64 matrix
        // instructions (the kernel slows down by what the vector instructions add).
        int px_img = 0, px_yo = 0, px_xo = 0;
        auto gload_px = [&](int c, int j) {
            float* fa = reinterpret_cast<float*>(pa);
            float* fb = reinterpret_cast<float*>(pb);
            const int p = c * XK + PX * wave_s + j;              // < 2^31 (checked by the caller)
            const bool pv = p < (int)n;
            if (j == 0) {
                const uint32_t pc = (uint32_t)min(p, (int)n - 1);
                const uint32_t img = fastdiv(pc, cp.div_img);
                const uint32_t rem = pc - img * (uint32_t)(cp.ho * cp.wo);
                const uint32_t yo = fastdiv(rem, cp.div_row);
                px_img = (int)img;
                px_yo = (int)yo;
                px_xo = (int)(rem - yo * (uint32_t)cp.wo);
            } else {
                ++px_xo;
                const bool wx = px_xo == cp.wo;
                px_xo = wx ? 0 : px_xo;
                px_yo += wx ? 1 : 0;
                const bool wy = px_yo == cp.ho;
                px_yo = wy ? 0 : px_yo;
                px_img += wy ? 1 : 0;
            }
            const int64_t origin = (((int64_t)px_img * cp.hp + px_yo * cp.stride) * cp.wp + px_xo * cp.stride) * cp.c;
            const float* __restrict__ win = X + (pv ? origin : cp.zero_origin);
#pragma unroll
            for (int q = 0; q < QN; ++q) {
                fa[q * PX + j] = win[offA[q]];
                if (load_b) fb[q * PX + j] = win[offB[q]];
            }
        };
        auto gload = [&](int c) {
            if (CONV) {
#pragma unroll
                for (int j = 0; j < PX; ++j) gload_px(c, j);
                return;
            }
            const int64_t k = (int64_t)c * XK + lk;
            if (FAST && k + 3 < n) {
#pragma unroll
                for (int u = 0; u < RG; ++u) {
                    pa[u] = *reinterpret_cast<const float4*>(arow[u] + k);
                    if (load_b) pb[u] = *reinterpret_cast<const float4*>(brow[u] + k);
                }
            } else {
#pragma unroll
                for (int u = 0; u < RG; ++u) {
                    float4 va = make_float4(0.f, 0.f, 0.f, 0.f), vb = va;
                    if (k + 0 < n) { va.x = arow[u][k + 0]; vb.x = brow[u][k + 0]; }
                    if (k + 1 < n) { va.y = arow[u][k + 1]; vb.y = brow[u][k + 1]; }
                    if (k + 2 < n) { va.z = arow[u][k + 2]; vb.z = brow[u][k + 2]; }
                    if (k + 3 < n) { va.w = arow[u][k + 3]; vb.w = brow[u][k + 3]; }
                    pa[u] = va;
                    pb[u] = vb;
                }
            }
        };
        auto sstore = [&](int buf) {
            if (CONV) {
                // PX consecutive pixels of a row: 16 bytes per store
#pragma unroll
                for (int q = 0; q < QN; ++q)
                    if (64 * q + 64 <= XT || lane + 64 * q < XT)
#pragma unroll
                        for (int x = 0; x < PX / 4; ++x) {
                            *reinterpret_cast<float4*>(&As[buf][lane + 64 * q][PX * wave + 4 * x]) = pa[q * PX / 4 + x];
                            if (load_b) *reinterpret_cast<float4*>(&Bs[buf][lane + 64 * q][PX * wave + 4 * x]) = pb[q * PX / 4 + x];
                        }
                return;
            }
#pragma unroll
            for (int u = 0; u < RG; ++u)
                if (RW * u + RW <= XT || lr + RW * u < XT) {
                    *reinterpret_cast<float4*>(&As[buf][lr + RW * u][lk]) = pa[u];
                    if (load_b) *reinterpret_cast<float4*>(&Bs[buf][lr + RW * u][lk]) = pb[u];
                }
        };

        double* __restrict__ out = Hpart + (int64_t)piece * d * d;
        // The pipeline over the piece's chunks; DG: diagonal tile of which only the MFMA tiles on and below
        // its diagonal are formed (XT = 128: 9 per wavefront instead of 16).
        auto run_piece = [&](auto dg_tag) {
            constexpr bool DG = decltype(dg_tag)::value;
            d4 acc[MT][MT];
            d4 accd[DG ? TK : 1];
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < MT; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int i = 0; i < (DG ? TK : 1); ++i) accd[i] = d4{0.0, 0.0, 0.0, 0.0};

            __syncthreads();              // LDS free (previous tile's last stage consumed)
            gload(chunk_at(0));
            sstore(0);
            __syncthreads();
            int cur = 0;
            for (int ci = 0; ci < len; ++ci) {
                const bool more = ci + 1 < len;
                // plain modes: 8 wide loads, issued up front.  Convolution mode: one pixel's loads per
                // group of 16 MFMAs (after the last chunk of a range the same chunk is simply loaded
                // again and not stored).
                const int cn = chunk_at(more ? ci + 1 : ci);
                if (!CONV && more) gload(cn);
#pragma unroll
                for (int g = 0; g < XK / 16; ++g) {
                    if constexpr (DG) {
                        auto after = [&](int ks) { if (CONV && g * 4 + ks < PX) gload_px(cn, g * 4 + ks); };
                        if (wave_s == 0) diag_mma<0, TB, TK>(As[cur], g, fr, fk, accd, after);
                        else if (wave_s == 1) diag_mma<1, TB, TK>(As[cur], g, fr, fk, accd, after);
                        else if (wave_s == 2) diag_mma<2, TB, TK>(As[cur], g, fr, fk, accd, after);
                        else if (NW == 4 || wave_s == 3) diag_mma<3, TB, TK>(As[cur], g, fr, fk, accd, after);
                        else if constexpr (NW == 8) {
                            if (wave_s == 4) diag_mma<4, TB, TK>(As[cur], g, fr, fk, accd, after);
                            else if (wave_s == 5) diag_mma<5, TB, TK>(As[cur], g, fr, fk, accd, after);
                            else if (wave_s == 6) diag_mma<6, TB, TK>(As[cur], g, fr, fk, accd, after);
                            else diag_mma<7, TB, TK>(As[cur], g, fr, fk, accd, after);
                        }
                    } else {
                        float4 fa[MT], fb[MT];
#pragma unroll
                        for (int i = 0; i < MT; ++i)
                            fa[i] = *reinterpret_cast<const float4*>(&As[cur][wm * WT + i * 16 + fr][g * 16 + fk]);
#pragma unroll
                        for (int j = 0; j < MT; ++j)
                            fb[j] = *reinterpret_cast<const float4*>(&Bs[cur][wn * WT + j * 16 + fr][g * 16 + fk]);
#pragma unroll
                        for (int ks = 0; ks < 4; ++ks) {
                            double a[MT], b[MT];
#pragma unroll
                            for (int i = 0; i < MT; ++i)
                                a[i] = (double)(ks == 0 ? fa[i].x : ks == 1 ? fa[i].y : ks == 2 ? fa[i].z : fa[i].w);
#pragma unroll
                            for (int j = 0; j < MT; ++j)
                                b[j] = (double)(ks == 0 ? fb[j].x : ks == 1 ? fb[j].y : ks == 2 ? fb[j].z : fb[j].w);
#pragma unroll
                            for (int i = 0; i < MT; ++i)
#pragma unroll
                                for (int j = 0; j < MT; ++j)
                                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
                            if (CONV && g * 4 + ks < PX) gload_px(cn, g * 4 + ks);
                        }
                    }
                }
                if (more) sstore(cur ^ 1);
                __syncthreads();
                cur ^= 1;
            }

            auto flush = [&](auto add_tag) {
                constexpr bool ADD = decltype(add_tag)::value;
                int fl = lane;
                asm volatile("" : "+v"(fl));       // addresses formed here, not kept over the pipeline
                auto put = [&](int gr, int gc, double v) {
                    if (gr >= d || gc >= d) return;
                    double* __restrict__ o = out + (int64_t)gr * d + gc;
                    *o = ADD ? *o + v : v;
                };
                if constexpr (DG) {
                    // wavefront w holds K consecutive MFMA tiles of the triangle: see TriOrder
#pragma unroll
                    for (int q = 0; q < TK; ++q) {
                        int sr, sc;
                        const bool mine = tri_place<TB>(wave_s * TK + q, sr, sc);
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (mine) put(i0 + sr * 16 + 4 * v + (fl >> 4), j0 + sc * 16 + (fl & 15), accd[q][v]);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < MT; ++i)
#pragma unroll
                        for (int j = 0; j < MT; ++j)
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                put(i0 + wm * WT + i * 16 + 4 * v + (fl >> 4), j0 + wn * WT + j * 16 + (fl & 15), acc[i][j][v]);
                }
            };
            if (fresh > 0) flush(std::false_type{});
            else flush(std::true_type{});
        };
        if constexpr (SINGLE) {
            run_piece(std::true_type{});
        } else if constexpr (LOWER) {
            if (diag) run_piece(std::true_type{});
            else run_piece(std::false_type{});
        } else {
            run_piece(std::false_type{});
        }

        // An accumulation's first launch finds nothing in its slabs and stores; where a tile has fewer pieces than the launch
        // has slabs (fresh), its workgroups put zeros into the others in turn.  (d = 512, 50176 columns, accumulate and
        // finalize: 295 us with a launch that clears 61 slabs and the sums read and written, 251 so.)
        if (fresh > 0) {
            const int64_t tile_last = tile_first + chunks - 1;
            int64_t last_range = (diag ? (tile_last + 1) * WD : diag_cost + (tile_last + 1 - diag_items) * 16) / range_cost;
            while (item_at(last_range * range_cost) > tile_last) --last_range;
            const int pieces = (int)(last_range - first_range) + 1;
            for (int p = piece + pieces; p < fresh; p += pieces) {
                double* __restrict__ rest = Hpart + (int64_t)p * d * d;
                for (int e = tid; e < XT * XT; e += 64 * NW) {
                    const int gr = i0 + e / XT, gc = j0 + e % XT;
                    if (gr < d && gc < d) rest[(int64_t)gr * d + gc] = 0.0;
                }
            }
        }
    }
}

// The split of a launch over n calibration columns: W ranges of equal cost over the items (tile, chunk),
// diagonal tiles first.  Cost units: 1/16 of a chunk of a tile below the diagonal (xxt_diag_cost for a
// diagonal tile's).
struct XxtPlan {
    int xt, nt, chunks, wgs;
    int64_t items;        // (tile, chunk) pairs
    int64_t range_cost;   // cost of one workgroup's range
};

static int64_t xxt_cost_per_chunk_column(int xt, int nt, int wd)     // cost of one chunk of every tile
{
    return (int64_t)wd * nt + 16 * ((int64_t)nt * (nt - 1) / 2);
}

// Number of d x d slabs of partial sums = the most pieces a tile can be cut into: a tile below the
// diagonal (the most expensive kind) spans at most ceil(its cost / range cost) ranges, plus one when it
// starts inside a range; the range cost is at least the total cost / W.
int xxt_pick_splits(int d)
{
    int most = 0;
    for (int xt : {xxt_base_tile(d), xxt_long_tile(d)}) {          // calls of either length fit
        const int nt = (d + xt - 1) / xt;
        const int64_t per_column = xxt_cost_per_chunk_column(xt, nt, xxt_diag_cost_min(xt));   // either mode fits
        most = std::max(most, (int)((16 * (int64_t)xxt_wgs(xt) + per_column - 1) / per_column) + 1);
    }
    return most;
}

static XxtPlan xxt_plan(int d, int64_t n, int splits, bool conv)
{
    XxtPlan p;
    p.xt = xxt_tile(d, n);
    p.nt = (d + p.xt - 1) / p.xt;
    p.chunks = (int)((n + XK - 1) / XK);
    p.items = ((int64_t)p.nt * (p.nt + 1) / 2) * p.chunks;
    const int64_t total_cost = xxt_cost_per_chunk_column(p.xt, p.nt, xxt_diag_cost(p.xt, conv)) * p.chunks;
    p.range_cost = (total_cost + xxt_wgs(p.xt) - 1) / xxt_wgs(p.xt);
    // a range must cost enough that no tile is cut into more than `splits` pieces
    const int64_t tile_cost = 16 * (int64_t)p.chunks;
    const int64_t min_cost = splits > 1 ? (tile_cost + splits - 2) / (splits - 1) : tile_cost;
    if (p.range_cost < min_cost) p.range_cost = min_cost;
    if (p.range_cost < 16) p.range_cost = 16;      // at least one whole chunk per range
    p.wgs = (int)((total_cost + p.range_cost - 1) / p.range_cost);
    return p;
}

// Slabs a launch over n calibration columns can write to (the rest of Hpart is not touched):
// a tile meets at most ceil(its cost / range cost) + 1 ranges.
int xxt_slabs_touched(int d, int64_t n, int splits, bool conv)
{
    const XxtPlan pl = xxt_plan(d, n, splits, conv);
    const int64_t p = (16 * (int64_t)pl.chunks + pl.range_cost - 1) / pl.range_cost + 1;
    return (int)(p < splits ? p : splits);
}

// Zero the part of the slabs [first, first + count) that the finalize kernels read, the lower triangle, whole tiles of 64 on the
// diagonal.  (A wider diagonal tile adds into entries above that part too; nothing reads those.)
__global__ __launch_bounds__(256) void clear_slabs_kernel(double* __restrict__ Hpart, int d, int first)
{
    const int a = blockIdx.x;
    const int lim = min(d, (a / 64 + 1) * 64);
    double* __restrict__ row = Hpart + ((int64_t)(first + blockIdx.y) * d + a) * d;
    for (int c = threadIdx.x; c < lim; c += 256) row[c] = 0.0;
}

hipError_t launch_clear_slabs(hipStream_t s, double* Hpart, int d, int first, int count)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(clear_slabs_kernel, dim3(d, count), dim3(256), 0, s, Hpart, d, first);
    return hipGetLastError();
}

template <int MODE>
static void xxt_launch(hipStream_t s, const XxtPlan& pl, const float* X, int64_t ld, int d, int64_t n, double* Hpart,
                       int splits, int fresh, const ConvP& cp, LaunchEvents ev)
{
    // pieces per tile (below the diagonal), rounded: the number of classes of ranges (see the kernel)
    const int64_t tile_cost = 16 * (int64_t)pl.chunks;
    int classes = (int)((tile_cost + pl.range_cost / 2) / pl.range_cost);
    classes = classes < 1 ? 1 : (classes > pl.wgs ? pl.wgs : classes);
    auto launch = [&](auto kernel) {
        hipExtLaunchKernelGGL(kernel, dim3(pl.wgs), dim3(64 * xxt_waves(pl.xt)), 0, s, ev.start, ev.stop, 0, X, ld, d, n, Hpart,
                              pl.chunks, pl.range_cost, pl.items, classes, splits, fresh, cp);
    };
    switch (pl.xt) {
    case 64: launch(xxt_kernel<MODE, 64>); break;
    case 96: launch(xxt_kernel<MODE, 96>); break;
    case 128: launch(xxt_kernel<MODE, 128>); break;
    default: launch(xxt_kernel<MODE, 160>); break;
    }
}

hipError_t launch_xxt(hipStream_t s, const float* X, int64_t ld, int d, int64_t n, double* Hpart, int splits, int fresh,
                      LaunchEvents ev)
{
    const XxtPlan pl = xxt_plan(d, n, splits, false);
    const bool fast = (ld % 4 == 0) && ((reinterpret_cast<uintptr_t>(X) & 15) == 0);
    ConvP none{};
    if (fast) xxt_launch<0>(s, pl, X, ld, d, n, Hpart, splits, fresh, none, ev);
    else      xxt_launch<1>(s, pl, X, ld, d, n, Hpart, splits, fresh, none, ev);
    return hipGetLastError();
}

// Convolution mode: padded = the copy written by launch_pad_maps ((n_img + 1) x hp x wp x c),
// d = c k^2, one calibration column per output pixel; npix = n_img * ho * wo < 2^31 - 64.
hipError_t launch_xxt_conv(hipStream_t s, const float* padded, int n_img, int hp, int wp, int c, int k, int stride,
                           int ho, int wo, int64_t npix, double* Hpart, int splits, int fresh,
                           LaunchEvents ev)
{
    const int d = c * k * k;
    const XxtPlan pl = xxt_plan(d, npix, splits, true);
    ConvP cp;
    cp.hp = hp; cp.wp = wp; cp.c = c; cp.k = k; cp.stride = stride; cp.ho = ho; cp.wo = wo;
    cp.zero_origin = (int64_t)n_img * hp * wp * c;
    cp.div_img = fastdiv_make((uint32_t)(ho * wo));
    cp.div_row = fastdiv_make((uint32_t)wo);
    cp.div_c = fastdiv_make((uint32_t)c);
    cp.div_k = fastdiv_make((uint32_t)k);
    xxt_launch<2>(s, pl, padded, 0, d, npix, Hpart, splits, fresh, cp, ev);
    return hipGetLastError();
}

// H[a][b] = H[b][a] = factor * sum_s Hpart[s][a][b]   for b <= a (lower slabs hold the sums)
// poison (may be null): a word that is non-zero when an input of the integer-slice path held an Inf or NaN;
// H then becomes NaN throughout, as the floating-point sum would have made the rows concerned.
// TURN: see store_symmetric.  ONE: the slabs one after another, not four in flight (launch_hessian_finalize).
template <bool ONE, bool TURN>
__global__ __launch_bounds__(256) void hessian_finalize_kernel(const double* __restrict__ Hpart, int splits, int sstride, int d,
                                                               double factor, double* __restrict__ H, double* __restrict__ H2,
                                                               const int* __restrict__ poison)
{
    if (blockIdx.x > blockIdx.y) return;
    const int b = blockIdx.x * 16 + (threadIdx.x & 15);
    const int a = blockIdx.y * 16 + (threadIdx.x >> 4);
    double s = 0.0;
    if (a < d && b <= a) {
        if (ONE)
            for (int k = 0; k < splits; ++k) s += Hpart[(int64_t)k * sstride * d * d + (int64_t)a * d + b];
        else
            s = slab_sum(Hpart + (int64_t)a * d + b, splits, (int64_t)sstride * d * d);
        s *= factor;
    }
    if (poison && *poison) s = __builtin_nan("");
    store_symmetric<TURN>(s, d, H, H2);
}

// Convolution mode: the slabs are in tap-major row order; H is written in (c, ky, kx) order.  ONE: the slabs one after another.  The
// gather takes a line of a slab for an entry or two, and finds it in the L2 again for the taps beside it only while all threads are
// at the same slab: with four of them in flight 576 columns (3 x 3) 58 -> 62 us for the call, 900 99 -> 103, 1200 (5 x 5) 130 -> 150.
// A slab of up to 256 columns stays in the L2 (147 columns 61 -> 60 us with four), and rows of a 1 x 1 kernel are read whole.
template <bool ONE, bool TURN>
__global__ __launch_bounds__(256) void hessian_finalize_conv_kernel(const double* __restrict__ Hpart, int splits, int sstride, int d,
                                                                    double factor, double* __restrict__ H, double* __restrict__ H2,
                                                                    int c, int kk, const int* __restrict__ poison)
{
    if (blockIdx.x > blockIdx.y) return;
    const int b = blockIdx.x * 16 + (threadIdx.x & 15);
    const int a = blockIdx.y * 16 + (threadIdx.x >> 4);
    double s = 0.0;
    if (a < d && b <= a) {
        const int ai = (a % kk) * c + a / kk, bi = (b % kk) * c + b / kk;
        const int hi = max(ai, bi), lo = min(ai, bi);
        if (ONE)
            for (int k = 0; k < splits; ++k) s += Hpart[(int64_t)k * sstride * d * d + (int64_t)hi * d + lo];
        else
            s = slab_sum(Hpart + (int64_t)hi * d + lo, splits, (int64_t)sstride * d * d);
        s *= factor;
    }
    if (poison && *poison) s = __builtin_nan("");
    store_symmetric<TURN>(s, d, H, H2);
}

// conv_c > 0: the slabs were accumulated in convolution mode with conv_c channels and conv_kk taps
// Small d, many slabs (a tile of a 64-column layer is cut into up to 1024 pieces): the lower triangles of groups of
// SLAB_GROUP consecutive slabs are first added into the first slab of each group, one workgroup per (16 x 16 entries,
// group), so that the finalize kernel -- one thread per entry, the slabs one after the other -- has SLAB_GROUP times
// fewer to walk through.  The order of the sum is fixed either way.
constexpr int SLAB_GROUP = 32;
__global__ __launch_bounds__(256) void hessian_group_slabs_kernel(double* __restrict__ Hpart, int splits, int d)
{
    const int b = blockIdx.x * 16 + (threadIdx.x & 15);
    const int a = blockIdx.y * 16 + (threadIdx.x >> 4);
    if (a >= d || b >= d || b > a) return;
    const int k0 = blockIdx.z * SLAB_GROUP, k1 = min(splits, k0 + SLAB_GROUP);
    const int64_t at = (int64_t)a * d + b;
    Hpart[(int64_t)k0 * d * d + at] = slab_sum(Hpart + (int64_t)k0 * d * d + at, k1 - k0, (int64_t)d * d);
}

hipError_t launch_hessian_finalize(hipStream_t s, double* Hpart, int splits, int d, double factor, double* H, double* H2,
                                   int conv_c, int conv_kk, const int* poison)
{
    dim3 grid((d + 15) / 16, (d + 15) / 16), block(256);
    int sstride = 1;
    if (splits > 2 * SLAB_GROUP) {
        const int groups = (splits + SLAB_GROUP - 1) / SLAB_GROUP;
        hipLaunchKernelGGL(hessian_group_slabs_kernel, dim3(grid.x, grid.y, groups), block, 0, s, Hpart, splits, d);
        splits = groups;
        sstride = SLAB_GROUP;
    }
    // Four slabs in flight where rows are read whole and a tile's pieces of them begin with a line or its half, or all slabs of a tile's
    // columns stay in the L2; else a line is found there again by the next tile only while all are at the same slab.  One after
    // another / four, the call: 288 x 900 21.9 / 16.8 us, 420 x 9000 59.0 / 54.2, 511 x 600 30.0 / 30.8, 512 x 20000 122.6 / 114.0, 701 x 900
    // 32.8 / 33.9, 520 of a 1 x 1 kernel 38.0 / 35.9, 640 x 500 29.9 / 28.9, 768 x 512 32.7 / 33.6, 896 x 700 43.5 / 44.3, 1040 x 512 48.2 / 45.0, 1400 x 700
    // 65.7 / 63.8; of few slabs 2048 x 512 71.5 / 72.1.
    const bool turn = d > 256, rows = conv_c <= 0 || conv_kk == 1;
    const bool four = d <= 256 || (rows && (d <= 504 || (d % 8 == 0 && (d <= 640 || (d >= 1000 && splits >= 8)))));
    if (conv_c > 0) {
        const auto kernel = !turn ? hessian_finalize_conv_kernel<false, false>
                          : four ? hessian_finalize_conv_kernel<false, true> : hessian_finalize_conv_kernel<true, true>;
        hipLaunchKernelGGL(kernel, grid, block, 0, s, Hpart, splits, sstride, d, factor, H, H2, conv_c, conv_kk, poison);
    } else {
        const auto kernel = !turn ? hessian_finalize_kernel<false, false> : four ? hessian_finalize_kernel<false, true> : hessian_finalize_kernel<true, true>;
        hipLaunchKernelGGL(kernel, grid, block, 0, s, Hpart, splits, sstride, d, factor, H, H2, poison);
    }
    return hipGetLastError();
}

}  // namespace fobq
