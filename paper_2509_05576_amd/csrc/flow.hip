// The two factorizations of the path as ONE launch each, by dependencies between 64 x 64 tiles instead of a launch per
// 64-column panel:
//   flow_inverse    H_d = R^T R (R = L^T), R^-T = L^-1 and Hinv = L^-T L^-1              (Section 5, item 1)
// A factorization is a chain of T = d / 64 diagonal blocks, each a few microseconds of sequential pivots, and between
// two of them only two tiles matter; everything else is product work that needs a fraction of the chip.  A launch per
// panel puts the launch gap, the loads and the recomputed panel products on that chain, and makes it wait for the
// slowest tile of every launch.
//
// Scheme.  A tile is computed once, left-looking: its owner (a workgroup of 8 wavefronts) adds up the products of all
// earlier panels in registers while their tiles become ready, finishes the tile with the block inverse of its own row
// and publishes it.  Workgroups take tiles from queues in a fixed order (a ticket each); whatever a tile waits for
// stands before it in its own queue, or in the queue served first, or is done by the workgroup that walks the chain
// (the first to start).  The earliest unfinished tile can therefore always proceed, however many workgroups are
// resident, and every wait ends.  (Should the device stop making progress all the same, every wait gives up after
// FLOW_MAX_POLLS looks, the launch drains and the call fails.)
//
// Exchange between compute units.  Each XCD has its own L2, which is not coherent with the others inside a launch.
// Everything that one workgroup hands to another during a launch goes through relaxed agent-scope atomic accesses
// (loads and stores that bypass the caches which are not shared): the producer stores a tile, waits until its stores
// are done, and sets the tile's word after a release fence; the consumer reads the word until it is set and loads.
// Measured: 1.85 us from the first store of a 32 KB tile to its last load on another XCD, and 16 TB/s when 256
// workgroups read tiles this way, against 9.6 TB/s that the products want at the full matrix rate.
#include <hip/hip_ext.h>

#include "tile_block.h"

namespace fobq {

constexpr int TILE = NB * NB;                        // doubles of a published tile
constexpr int FLOW_LDS = SWEEP_LDS + 4 * NB * DL;    // doubles: two double-buffered operand tiles, or the chain's blocks
constexpr int FLOW_MAX_POLLS = 1 << 22;              // several seconds
// words of a launch, all zero before it: counters, then one word per tile (T x T), then two per diagonal block for the
// sums that are handed to the chain
enum { FW_ROLE = 0, FW_QUEUE1 = 1, FW_QUEUE2 = 2, FW_ABORT = 3, FW_HEAD = 16 };

__device__ __forceinline__ double ld_shared(const double* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_shared(double* p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ int ld_word(const int* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_word(int* p, int v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// what both launches have: d columns in T blocks; tiles: T x T published tiles, [row of tiles][column of tiles][64][64];
// gt: T tiles, the transposed block inverses, then T tiles for the sums D(k, 0) (see Queue1); stalled: status word for a launch that gave up
struct FlowP {
    int d, T, n1;        // n1: workgroups that serve queue 1 first (the chain's workgroup not counted)
    int* words;
    double* tiles;
    double* gt;
    int* notpd;
    int* stalled;
};

__device__ __forceinline__ double* tile_at(const FlowP& f, int i, int j) { return f.tiles + ((int64_t)i * f.T + j) * TILE; }
__device__ __forceinline__ int* tile_word(const FlowP& f, int i, int j) { return f.words + FW_HEAD + i * f.T + j; }
__device__ __forceinline__ int* hand_word(const FlowP& f, int k, int which) { return f.words + FW_HEAD + f.T * f.T + 2 * k + which; }
__device__ __forceinline__ double* hand_tile(const FlowP& f, int k) { return f.gt + (int64_t)(f.T + k) * TILE; }
static int flow_words(int T) { return FW_HEAD + T * T + 2 * T; }

// One wavefront: waits until the word of every lane that has one is set.
__device__ __forceinline__ void flow_wait(const FlowP& f, const int* word, bool has)
{
    for (int n = 0;; ++n) {
        const int v = has ? ld_word(word) : 1;
        if (__all(v != 0)) break;
        if (n >= FLOW_MAX_POLLS) st_word(f.words + FW_ABORT, 1);
        if ((n & 31) == 31 && ld_word(f.words + FW_ABORT) != 0) break;
        __builtin_amdgcn_s_sleep(1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");    // (keeps the loads that follow behind the last look)
}

// All threads: what the workgroup has stored with st_shared is visible before the word is set.
__device__ __forceinline__ void flow_publish(int* word)
{
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        st_word(word, 1);
    }
}

// Operand tiles in LDS: rows of 64 doubles, the two halves of 32 banks exchanged in odd rows, so that the fragment reads
// of a half wavefront (16 columns of two neighbouring rows) meet no bank conflict.
__device__ __forceinline__ int swz(int row, int col) { return row * 64 + (col ^ ((row & 1) << 4)); }

// c -= sum_{q0 <= q < q1} A_q^T B_q, A_q and B_q published 64 x 64 tiles [k][m], [k][n]; c in the accumulator layout: rows
// wr * 16 + 4 v + fq, columns w2 * 32 + 16 j + fr of wavefront (wr, w2).  src.a(q), src.b(q): the tiles, src.wa(q),
// src.wb(q): their words.  The loads of the next two steps are in flight during the products of a step as far as their
// tiles are known to be ready (under load a tile takes longer to arrive than the 1.7 us of a step's products); what is
// not known to be ready is looked for when its turn comes.  LDS: four tiles, one barrier per step.
template <class Src>
__device__ __forceinline__ void flow_sum(const FlowP& f, double* lds, const Src& src, int q0, int q1, d4 (&c)[2])
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
    int known = q0, loaded = q0;         // the tiles of the steps before `known` are ready, those before `loaded` on their way
    auto look = [&](int q) {             // wavefront-uniform
        for (int n = 0;; ++n) {
            const int s = min(q + (lane & 31), q1 - 1);
            const unsigned long long m = __ballot(ld_word(lane < 32 ? src.wa(s) : src.wb(s)) != 0);
            const unsigned both = (unsigned)m & (unsigned)(m >> 32);
            const int k = both == ~0u ? 32 : __builtin_ctz(~both);
            if (k > 0) { known = min(q + k, q1); break; }
            if (n >= FLOW_MAX_POLLS) st_word(f.words + FW_ABORT, 1);
            if ((n & 31) == 31 && ld_word(f.words + FW_ABORT) != 0) { known = q1; break; }
            __builtin_amdgcn_s_sleep(1);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    };
    auto load = [&](double (&pa)[8], double (&pb)[8]) {      // step `loaded`
        const double* a = src.a(loaded) + wave * 512 + lane;
        const double* b = src.b(loaded) + wave * 512 + lane;
#pragma unroll
        for (int u = 0; u < 8; ++u) { pa[u] = ld_shared(a + u * 64); pb[u] = ld_shared(b + u * 64); }
        ++loaded;
    };
    auto step = [&](int q, double* As, double (&pa)[8], double (&pb)[8], double (&na)[8], double (&nb)[8]) {
        double* Bs = As + TILE;
        if (loaded == q) {
            look(q);
            load(pa, pb);
        }
        const int w0 = here(wave * 512 + lane), w1 = here(wave * 512 + (lane ^ 16));
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            As[(u & 1 ? w1 : w0) + u * 64] = pa[u];
            Bs[(u & 1 ? w1 : w0) + u * 64] = pb[u];
        }
        __syncthreads();
        if (loaded == q + 1 && q + 1 < known) load(na, nb);
        if (loaded == q + 2 && q + 2 < known) load(pa, pb);
        const int ra = here(swz(fq, wr * 16 + fr)), rb = here(swz(fq, w2 * 32 + fr)), rc = here(swz(fq, w2 * 32 + 16 + fr));
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) {
            const double a = -As[ra + ks * 256];
            c[0] = mfma4(a, Bs[rb + ks * 256], c[0]);
            c[1] = mfma4(a, Bs[rc + ks * 256], c[1]);
        }
    };
    double pa[8], pb[8], na[8], nb[8];
    int q = q0;
    for (; q + 1 < q1; q += 2) {
        step(q, lds, pa, pb, na, nb);
        step(q + 1, lds + 2 * TILE, na, nb, pa, pb);
    }
    if (q < q1) step(q, lds, pa, pb, na, nb);
}

// u = G c for the finished sum c of a tile in row i of tiles, G = the block inverse of that row (its transpose is
// gt[i]).  u: row tiles {w2, 3 - w2} (G is lower triangular: 20 of 32 (k-step, tile) pairs either way), columns
// wr * 16 ..  steps: how many the sum had (the product takes the pair of LDS tiles that its last step did not read).
template <int W>
__device__ __forceinline__ void flow_tri_product(const double* Gs, const double* Cs, int wr, int fr, int fq, d4 (&u)[2])
{
    const int rc = here(swz(fq, wr * 16 + fr)), r0 = here(swz(fq, W * 16 + fr)), r1 = here(swz(fq, (3 - W) * 16 + fr));
#pragma unroll
    for (int ks = 0; ks < 16 - 4 * W; ++ks) {
        const double b = Cs[rc + ks * 256];
        if (ks < 4 * W + 4) u[0] = mfma4(Gs[r0 + ks * 256], b, u[0]);
        u[1] = mfma4(Gs[r1 + ks * 256], b, u[1]);
    }
}

__device__ __forceinline__ void flow_row_product(const FlowP& f, double* lds, int i, int steps, const d4 (&c)[2], d4 (&u)[2])
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
    double* Gs = lds + (steps & 1) * 2 * TILE;
    double* Cs = Gs + TILE;
    flow_wait(f, tile_word(f, i, i), lane == 0);
    const double* g = f.gt + (int64_t)i * TILE + wave * 512 + lane;
    double pg[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) pg[x] = ld_shared(g + x * 64);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) Cs[here(swz(wr * 16 + fq, w2 * 32 + 16 * j + fr)) + v * 256] = c[j][v];
    const int w0 = here(wave * 512 + lane), w1 = here(wave * 512 + (lane ^ 16));
#pragma unroll
    for (int x = 0; x < 8; ++x) Gs[(x & 1 ? w1 : w0) + x * 64] = pg[x];
    __syncthreads();
    u[0] = d4{0.0, 0.0, 0.0, 0.0};
    u[1] = d4{0.0, 0.0, 0.0, 0.0};
    if (w2 == 0) flow_tri_product<0>(Gs, Cs, wr, fr, fq, u);
    else flow_tri_product<1>(Gs, Cs, wr, fr, fq, u);
}

// Queue 1 of both launches, in the order of the rows of tiles: the sums D(1, .) first, then for every row p the tile
// (p, p + 2), the sums D(p + 2, .) of the diagonal block two further on, and the tiles (p, p + 3), (p, p + 4), ...
// D(k, 0) / D(k, 1) = tile (k - 1, k) / (k, k) with the panels before k - 1 taken off; the chain does the rest.  (They are
// handed over in a tile of their own and in the place of tile (k, k); the chain's workgroup has read all of the latter before it
// stores tile (k, k), but its wavefronts store tile (k - 1, k) while others still read D(k, 0).)
struct Queue1Item { int kind, i, j; };               // kind 0: tile (i, j); 1: D(i, j)
struct Queue1 {
    int p = 0, base = 2;                             // row of tiles of the last ticket, its first ticket
    __device__ __forceinline__ Queue1Item at(int t, int T)
    {
        if (t < 2) return {1, 1, t};
        while (t - base >= T - p) { base += T - p; ++p; }
        const int u = t - base;
        if (u == 0) return {0, p, p + 2};
        if (u < 3) return {1, p + 2, u - 1};
        return {0, p, p + u};
    }
};
__device__ __forceinline__ int queue1_length(int T) { return T < 2 ? 0 : T < 3 ? 2 : T * (T + 1) / 2 - 1; }

// the next ticket of a queue, for the whole workgroup (slot: a word of LDS)
__device__ __forceinline__ int flow_ticket(const FlowP& f, int queue, int* slot)
{
    __syncthreads();                                 // the LDS of the tile before is free, the slot has been read
    if (threadIdx.x == 0) *slot = __hip_atomic_fetch_add(f.words + queue, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    return *slot;
}

// ---------------------------------------------------------------------------
// H_d = R^T R in the upper tiles, X = R^-T (= L^-1) in the lower ones, Hinv = X^T X.
//   R_ij = G_i (H_ij - sum_{q < i} R_qi^T R_qj), i < j;   G_i = R_ii^-T from chol_block
//   X_ij = G_i (    - sum_{j <= q < i} R_qi^T X_qj), j < i;  X_ii = G_i
//   Hinv_mn = sum_{k >= n} X_km^T X_kn, m <= n
// Queue 1: R.  Queue 2: X row by row, then Hinv with the longest sums first (they need all of X and are the only work
// left after the chain has ended).
struct FlowInverseP {
    FlowP f;
    const double* H;
    double damp, damp_abs;
    double* Hinv;          // d x d: the tiles on and above the diagonal are written
};

// lambda = damp * mean(diag H) + damp_abs: by every workgroup that needs it, in the same order
__device__ __forceinline__ double flow_lambda(const FlowInverseP& p, double* part)
{
    const int tid = threadIdx.x;
    double s = 0.0;
    for (int a = tid; a < p.f.d; a += NT) s += p.H[(int64_t)a * p.f.d + a];
    __syncthreads();
    part[tid] = s;
    __syncthreads();
    for (int w = NT / 2; w > 0; w >>= 1) {
        if (tid < w) part[tid] += part[tid + w];
        __syncthreads();
    }
    const double lam = p.damp * (part[0] / (double)p.f.d) + p.damp_abs;
    __syncthreads();
    return lam;
}

// tile (i, j) of H (0 past d) in the accumulator layout, lambda added on the diagonal
__device__ __forceinline__ void flow_init_h(const FlowInverseP& p, int i, int j, double lam, d4 (&c)[2])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
    const int d = p.f.d;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int gm = NB * i + wr * 16 + 4 * v + fq, gn = NB * j + w2 * 32 + 16 * h + fr;
            double x = (gm < d && gn < d) ? p.H[(int64_t)gm * d + gn] : 0.0;
            if (gm == gn) x += lam;
            c[h][v] = x;
        }
}

struct SumR {      // R_qi^T R_qj
    FlowP f; int i, j;
    __device__ const double* a(int q) const { return tile_at(f, q, i); }
    __device__ const double* b(int q) const { return tile_at(f, q, j); }
    __device__ const int* wa(int q) const { return tile_word(f, q, i); }
    __device__ const int* wb(int q) const { return tile_word(f, q, j); }
};

// The chain: the workgroup that walks the diagonal blocks.  For block k it takes the sums D(k, 0), D(k, 1), finishes
// tile (k - 1, k) with the inverse of the block before (still in its LDS), publishes it, takes its product off the
// diagonal block, factors that and publishes the block inverse.  Everything else hides behind other workgroups, so
// this is written for latency: D(k, 0) is loaded as MFMA operands, without a stage in LDS; the loads of D(k, .) are on
// their way while the stores of the block inverse drain, when a look says that they are ready; of the diagonal block
// only the tiles of its triangle are formed, and only the first 16 columns' before the first sweep starts (two of the
// other six are formed beside it).
// A wavefront's 16 x 16 tiles of the diagonal block (row tile >= column tile): one before the first sweep, wavefronts
// 1 and 2 one more during it.
__device__ __forceinline__ void chain_tiles(int wave, int (&rt)[2], int (&ct)[2])
{
    rt[0] = wave < 4 ? wave : wave == 4 ? 1 : wave == 6 ? 3 : 2;
    ct[0] = wave < 4 ? 0 : wave == 7 ? 2 : 1;
    rt[1] = 3;
    ct[1] = wave == 1 ? 2 : 3;
}

// The block inverse G (lower triangular, DL-strided in LDS) as A operand of the row tiles {W, 3 - W}: row tile t needs the
// k-steps 0 .. 4 t + 3 only, 20 of 32 (k-step, tile) pairs for either W: g[0 .. 4 W + 3] are tile W's, the rest 3 - W's.
template <int W>
__device__ __forceinline__ void chain_load_inverse(const double* Xm, int fr, int fq, double (&g)[20])
{
    const int r0 = here((W * 16 + fr) * DL + fq), r1 = here(((3 - W) * 16 + fr) * DL + fq);
#pragma unroll
    for (int x = 0; x < 20; ++x) {
        const bool lo = x < 4 * W + 4;
        g[x] = Xm[(lo ? r0 : r1) + 4 * (lo ? x : x - 4 * W - 4)];
    }
}

template <int W>
__device__ __forceinline__ void chain_row_product(const double (&g)[20], const double (&vb)[16], d4 (&u)[2])
{
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
        if (ks < 4 * W + 4) u[0] = mfma4(g[ks], vb[ks], u[0]);
        if (ks < 16 - 4 * W) u[1] = mfma4(g[4 * W + 4 + ks], vb[ks], u[1]);
    }
}

__device__ __forceinline__ void flow_chain_inverse(const FlowInverseP& p, double* lds)
{
    const FlowP& f = p.f;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
    double* Am = lds + SWEEP_LDS;
    double* Xm = Am + NB * DL;
    double* Vs = Xm + NB * DL;
    int rt[2], ct[2];
    chain_tiles(wave, rt, ct);
    const bool second = wave == 1 || wave == 2;
    const int t[2] = {w2, 3 - w2};               // row tiles of the product with the block inverse
    d4 c[2];
    double vb[16], g[20];
    auto load_sums = [&](int k) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        const double* V = hand_tile(f, k) + fq * 64 + wr * 16 + fr;
        const double* D = tile_at(f, k, k) + fq * 64 + fr;
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) vb[ks] = ld_shared(V + ks * 256);
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (h == 0 || second) {
#pragma unroll
                for (int v = 0; v < 4; ++v) c[h][v] = ld_shared(D + (rt[h] * 16 + 4 * v) * 64 + ct[h] * 16);
            }
    };
    auto store_diag = [&](int h, int nb) {
        const int at = here((rt[h] * 16 + fq) * DL + ct[h] * 16 + fr);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int m = rt[h] * 16 + 4 * v + fq, n = ct[h] * 16 + fr;
            Am[at + 4 * v * DL] = c[h][v];
            if (nb < NB && (m >= nb || n >= nb)) Am[m * DL + n] = m == n ? 1.0 : 0.0;     // identity padding past d
        }
    };
    auto diag_product = [&](int h) {             // c[h] -= R_{k-1,k}[:, row tile]^T R_{k-1,k}[:, column tile]
        const int ra = here(swz(fq, rt[h] * 16 + fr)), rb = here(swz(fq, ct[h] * 16 + fr));
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) c[h] = mfma4(-Vs[ra + ks * 256], Vs[rb + ks * 256], c[h]);
    };
    // chol_block writes the lower triangle of the inverse, whole 16 x 16 tiles on the diagonal included (zeros above it);
    // the tiles above stay as they are.  (Past d the last block's inverse is the identity: its rows meet zeros only.)
    for (int x = tid; x < NB * NB; x += NT) Xm[(x >> 6) * DL + (x & 63)] = 0.0;
    bool have = false;                           // the sums of the next block are loaded
    for (int k = 0; k < f.T; ++k) {
        const int nb = min(NB, f.d - NB * k);
        if (k == 0) {
            const double lam = flow_lambda(p, Am);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int m = rt[h] * 16 + 4 * v + fq, n = ct[h] * 16 + fr;
                    c[h][v] = (m < nb && n < nb) ? p.H[(int64_t)m * f.d + n] : 0.0;
                    if (m == n) c[h][v] += lam;
                }
        } else {
            if (!have) {
                flow_wait(f, hand_word(f, k, lane & 1), lane < 2);
                load_sums(k);
            }
            // R_{k-1,k} = G D(k, 0): row tiles t, columns wr * 16 ..
            d4 u[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
            if (w2 == 0) chain_row_product<0>(g, vb, u);
            else chain_row_product<1>(g, vb, u);
            double* R = tile_at(f, k - 1, k);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int m = t[i] * 16 + 4 * v + fq, n = wr * 16 + fr;
                    Vs[here(swz(t[i] * 16 + fq, n)) + v * 256] = u[i][v];
                    st_shared(R + m * 64 + n, u[i][v]);
                }
            __syncthreads();
            diag_product(0);
            __builtin_amdgcn_s_waitcnt(0);
        }
        store_diag(0, nb);
        __syncthreads();
        if (k > 0 && tid == NT - 64) {           // a wavefront that the sweeps leave idle
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            st_word(tile_word(f, k - 1, k), 1);
        }
        int seen = 1;                            // words of the next block's sums, looked at while the last sweep runs
        chol_block(Am, Xm, lds, f.notpd, [&]() {
            if (second) {
                if (k > 0) diag_product(1);
                store_diag(1, nb);
            }
        }, [&]() {
            if (lane < 2 && k + 1 < f.T) seen = ld_word(hand_word(f, k + 1, lane));
        });
        // the next block's sums: looked for before and after the stores of the block inverse
        have = k + 1 < f.T && __all(seen != 0);
        if (have) load_sums(k + 1);
        double* Gt = f.gt + (int64_t)k * TILE;
        double* G = tile_at(f, k, k);
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            const int y = wave * 8 + x;
            st_shared(Gt + y * 64 + lane, Xm[lane * DL + y]);
            st_shared(G + y * 64 + lane, Xm[y * DL + lane]);
        }
        if (k + 1 < f.T) {
            if (!have) {
                have = __all(lane < 2 ? ld_word(hand_word(f, k + 1, lane)) != 0 : true);
                if (have) load_sums(k + 1);
            }
            if (w2 == 0) chain_load_inverse<0>(Xm, fr, fq, g);
            else chain_load_inverse<1>(Xm, fr, fq, g);
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (tid == NT - 64) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            st_word(tile_word(f, k, k), 1);
        }
    }
}

__global__ __launch_bounds__(NT, 2) void flow_inverse_kernel(FlowInverseP p)
{
    __shared__ double lds[FLOW_LDS];
    __shared__ int slot;
    const FlowP& f = p.f;
    const int T = f.T;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
    double* tiles = lds + SWEEP_LDS;
    const int role = flow_ticket(f, FW_ROLE, &slot);
    if (role == 0) flow_chain_inverse(p, lds);
    else if (role <= f.n1) {
        Queue1 q1;
        const int n = queue1_length(T);
        for (;;) {
            const int t = flow_ticket(f, FW_QUEUE1, &slot);
            if (t >= n) break;
            const Queue1Item it = q1.at(t, T);
            d4 c[2], u[2];
            if (it.kind == 0) {
                flow_init_h(p, it.i, it.j, 0.0, c);
                flow_sum(f, tiles, SumR{f, it.i, it.j}, 0, it.i, c);
                flow_row_product(f, tiles, it.i, it.i, c, u);
                double* out = tile_at(f, it.i, it.j);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int v = 0; v < 4; ++v) st_shared(out + ((h ? 3 - w2 : w2) * 16 + 4 * v + fq) * 64 + wr * 16 + fr, u[h][v]);
                flow_publish(tile_word(f, it.i, it.j));
            } else {
                const int k = it.i, ti = it.j ? k : k - 1;
                const double lam = it.j ? flow_lambda(p, tiles) : 0.0;
                flow_init_h(p, ti, k, lam, c);
                flow_sum(f, tiles, SumR{f, ti, k}, 0, k - 1, c);
                double* out = it.j ? tile_at(f, k, k) : hand_tile(f, k);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int v = 0; v < 4; ++v) st_shared(out + (wr * 16 + 4 * v + fq) * 64 + w2 * 32 + 16 * h + fr, c[h][v]);
                flow_publish(hand_word(f, k, it.j));
            }
        }
    }
    const int nx = T * (T - 1) / 2, nh = T * (T + 1) / 2;
    for (;;) {
        const int t = flow_ticket(f, FW_QUEUE2, &slot);
        if (t >= nx + nh) break;
        d4 c[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}}, u[2];
        if (t < nx) {
            int i, j;
            tri_decode(t, i, j);
            ++i;
            flow_sum(f, tiles, SumR{f, i, j}, j, i, c);          // tile (q, j), q >= j, is X_qj
            flow_row_product(f, tiles, i, i - j, c, u);
            double* out = tile_at(f, i, j);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int v = 0; v < 4; ++v) st_shared(out + ((h ? 3 - w2 : w2) * 16 + 4 * v + fq) * 64 + wr * 16 + fr, u[h][v]);
            flow_publish(tile_word(f, i, j));
        } else {
            int m, n;
            tri_decode(t - nx, n, m);
            flow_sum(f, tiles, SumR{f, m, n}, n, T, c);          // X_km^T X_kn, k >= n >= m
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int gm = NB * m + wr * 16 + 4 * v + fq, gn = NB * n + w2 * 32 + 16 * h + fr;
                    if (gm < f.d && gn < f.d) p.Hinv[(int64_t)gm * f.d + gn] = -c[h][v];
                }
        }
    }
    if (threadIdx.x == 0 && ld_word(f.words + FW_ABORT) != 0) *f.stalled = 1;
}

int64_t flow_inverse_words(int d) { return flow_words((d + NB - 1) / NB); }
size_t flow_tiles_bytes(int d) { const size_t T = (d + NB - 1) / NB; return T * T * TILE * sizeof(double); }
size_t flow_gt_bytes(int d) { const size_t T = (d + NB - 1) / NB; return 2 * T * TILE * sizeof(double); }

hipError_t launch_flow_inverse(hipStream_t s, int cus, const double* H, int d, double damp, double damp_abs, double* Hinv, double* tiles,
                               double* gt, int* words, int* notpd, int* stalled)
{
    FlowInverseP p;
    p.f.d = d;
    p.f.T = (d + NB - 1) / NB;
    const int T = p.f.T;
    // One workgroup per compute unit at most (its LDS), no more than there are tiles in flight.
    const int64_t total = 1 + 2 * (int64_t)T * T;
    const int wgs = (int)(total < cus ? total : cus);
    p.f.n1 = 2 * T < wgs / 2 ? 2 * T : wgs / 2;
    if (p.f.n1 < 1) p.f.n1 = 1;
    p.f.words = words; p.f.tiles = tiles; p.f.gt = gt; p.f.notpd = notpd; p.f.stalled = stalled;
    p.H = H; p.damp = damp; p.damp_abs = damp_abs; p.Hinv = Hinv;
    hipLaunchKernelGGL(flow_inverse_kernel, dim3(wgs), dim3(NT), 0, s, p);
    return hipGetLastError();
}

}  // namespace fobq
