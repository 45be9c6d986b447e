// The two factorizations of the path as ONE launch each, by dependencies between 64 x 64 tiles instead of a launch per
// 64-column panel:
//   flow_inverse    H_d = R^T R (R = L^T), R^-T = L^-1 and Hinv = L^-T L^-1              (Section 5, item 1)
//   flow_eliminate  the shared-Hinv elimination with the column loop that follows it     (Eq. 8, 9, 12, Section 4.2)
// and of several small layers at once (the *_batch kernels: the same bodies, each workgroup on one layer).
// A factorization is a chain of T = d / 64 diagonal blocks, each a few microseconds of sequential pivots, and between
// two of them only two tiles matter; everything else is product work that needs a fraction of the chip.  A launch per
// panel puts the launch gap, the loads and the recomputed panel products on that chain, and makes it wait for the
// slowest tile of every launch.
//
// Scheme.  A tile is computed once, left-looking: its owner (a workgroup of 8 wavefronts) adds up the products of all
// earlier panels in registers while their tiles become ready, finishes the tile with the block inverse of its own row
// and publishes it.  Workgroups take tiles from queues in a fixed order (a ticket each).  All the work of a launch has one
// order in which whatever a tile waits for stands before it; each queue is a part of that order, and the workgroup that
// walks the chain is the first to start, the next ones serve one queue each.  So the earliest unfinished tile has its
// workgroup as soon as one workgroup per queue is resident, it can always proceed, and every wait ends.  (Should a launch stop
// all the same -- nobody draws a ticket for three quarters of a minute, see flow_gives_up -- its waits give up, it drains and the call
// fails.  A wait may be as long as it likes while tickets are drawn: foreign work on the device only delays it.)
//
// Exchange between compute units.  Each XCD has its own L2, which is not coherent with the others inside a launch.
// Everything that one workgroup hands to another during a launch goes through relaxed agent-scope atomic accesses
// (loads and stores that bypass the caches which are not shared): the producer stores a tile, waits until its stores
// are done, and sets the tile's word; the consumer reads the word until it is set and loads.  Stores that are done are
// where every compute unit finds them, and nothing else crosses, so the word needs no release at agent scope in front of it:
// that writes the XCD's whole L2 back, for every tile of every workgroup (4.76 against 4.61 ms for a layer of 2048 x 4608, 1046 against
// 990 us for 1000 x 2048).
// Measured with a kernel that does nothing else: 1.85 us from the first store of a 32 KB tile to its last load by a workgroup on
// another XCD, and 16 TB/s when 256 workgroups read published tiles this way, against 9.6 TB/s that the products want at the
// full matrix rate.
// Registers: the inverse 192 VGPRs; the elimination, with the chain, the tiles and the column parts in one body, 199, and 145 to
// 155 SGPRs kept in lanes of vector registers (no scratch in either).
#include <string.h>

#include <algorithm>

#include "column_chain.h"
#include "tile_block.h"

namespace fobq {

constexpr int TILE = NB * NB;                        // doubles of a published tile
constexpr int FLOW_LDS = SWEEP_LDS + 4 * NB * DL;    // doubles: two double-buffered operand tiles, or the chain's blocks
// words of a launch, all zero before it: counters, then one word per tile (T x T), then three per diagonal block: for the two
// sums that are handed to the chain and for the sum of tile (k - 2, k) that goes into them
enum { FW_ROLE = 0, FW_QUEUE1 = 1, FW_QUEUE2 = 2, FW_QUEUE3 = 3, FW_ABORT = 4, FW_HEAD = 16 };

__device__ __forceinline__ double ld_shared(const double* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_shared(double* p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ int ld_word(const int* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_word(int* p, int v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// what both launches have: d columns in T blocks; tiles: T x T published tiles, [row of tiles][column of tiles][64][64];
// gt: T tiles, the transposed block inverses, then T tiles for the sums D(k, 0) (see Queue1), then T for
// those of tiles (k - 2, k) (sum_tile); stalled: status word for a launch that gave up
struct FlowP {
    int d, T;
    int n1, n2, n3;      // workgroups that serve queue 1 / 2 / 3 first (the chain's workgroup not counted)
    int looks;           // see flow_gives_up
    int* words;
    double* tiles;
    double* gt;
    int* notpd;
    int* stalled;
};

__device__ __forceinline__ double* tile_at(const FlowP& f, int i, int j) { return f.tiles + ((int64_t)i * f.T + j) * TILE; }
__device__ __forceinline__ int* tile_word(const FlowP& f, int i, int j) { return f.words + FW_HEAD + i * f.T + j; }
__device__ __forceinline__ int* hand_word(const FlowP& f, int k, int which) { return f.words + FW_HEAD + f.T * f.T + 3 * k + which; }
__device__ __forceinline__ double* hand_tile(const FlowP& f, int k) { return f.gt + (int64_t)(f.T + k) * TILE; }
__device__ __forceinline__ double* sum_tile(const FlowP& f, int k) { return f.gt + (int64_t)(2 * f.T + k) * TILE; }
static int flow_words(int T) { return FW_HEAD + T * T + 3 * T; }

// One wavefront, after a look that found nothing: whether to stop waiting.  n counts the looks since the launch was last seen
// to move, that is to draw tickets (roles or tiles: whoever finishes a tile draws the next); after f.looks of them the
// launch is given up, for all its wavefronts.  seen: the counters at the last check (per lane; both start as in FlowPatience).
struct FlowPatience { int n = 0, seen = -1; };
__device__ __forceinline__ bool flow_gives_up(const FlowP& f, FlowPatience& w)
{
    ++w.n;
    if ((w.n & 31) == 0 || w.n >= f.looks) {
        const int lane = threadIdx.x & 63;
        const int v = ld_word(f.words + min(lane, (int)FW_ABORT));
        if (__builtin_amdgcn_readlane(v, FW_ABORT) != 0) return true;
        if (__any(lane < FW_ABORT && v != w.seen)) w.n = 0;
        else if (w.n >= f.looks) {
            st_word(f.words + FW_ABORT, 1);
            return true;
        }
        w.seen = v;
    }
    __builtin_amdgcn_s_sleep(1);
    return false;
}

// One wavefront: waits until the word of every lane that has one is set.
__device__ __forceinline__ void flow_wait(const FlowP& f, const int* word, bool has)
{
    for (FlowPatience w;;) {
        const int v = has ? ld_word(word) : 1;
        if (__all(v != 0) || flow_gives_up(f, w)) break;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");    // (keeps the loads that follow behind the last look)
}

// All threads: what the workgroup has stored with st_shared or st_pair is visible before the word is set.
__device__ __forceinline__ void flow_publish(int* word)
{
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        st_word(word, 1);
    }
}

// Operand tiles [k][m] in LDS: two rows interleaved, element (k, m) at (k / 2) * 128 + 2 m + (k & 1), so that a fragment read is
// 16 bytes -- the elements of two MFMAs, the first of rows k = 8 kk + 2 fq, the second of the rows after them -- and meets no
// bank conflict, and a lane that holds two rows of a column stores 16 bytes.
typedef double d2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int pair_at(int k, int m) { return (k >> 1) * 128 + 2 * m + (k & 1); }
__device__ __forceinline__ d2& pair(double* p) { return *reinterpret_cast<d2*>(p); }
__device__ __forceinline__ const d2& pair(const double* p) { return *reinterpret_cast<const d2*>(p); }
// Published tiles are laid out the same way in memory, so that a lane moves 16 bytes at a time: rows k and k + 1 (k even) of a
// column.  They are read and written past the caches that are not shared (bit 4: sc1), as ld_shared and st_shared do.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_buffer(const double* tile)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(tile), 0, TILE * (int)sizeof(double), 0x00020000);
}
__device__ __forceinline__ d2 ld_pair(const double* tile, int at)
{
    return __builtin_bit_cast(d2, __builtin_amdgcn_raw_buffer_load_b128(tile_buffer(tile), at * 8, 0, 16));
}
__device__ __forceinline__ void st_pair(double* tile, int at, d2 v)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), tile_buffer(tile), at * 8, 0, 16);
}
// Rows m0 + 4 v + fq (v = 0 .. 3) of column n in a tile, from the accumulator layout: lanes fq and fq + 1 (fq even) hold the rows
// of a pair, and exchange what makes two pairs of theirs whole.
__device__ __forceinline__ void st_rows(double* tile, int m0, int n, int fq, const d4& x)
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(x[2 * i]), __double2loint(x[2 * i + 1]), false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x[2 * i]), __double2hiint(x[2 * i + 1]), false, false);
        const d2 y = {__hiloint2double(hi[0], lo[0]), __hiloint2double(hi[1], lo[1])};
        st_pair(tile, ((m0 >> 1) + 4 * i + 2 * (fq & 1) + (fq >> 1)) * 128 + 2 * n, y);
    }
}
// the chain's tiles (8-byte reads): rows of 64 doubles, the two halves of 32 banks exchanged in odd rows
__device__ __forceinline__ int swz(int row, int col) { return row * 64 + (col ^ ((row & 1) << 4)); }

// c += sum_{q0 <= q < q1} A_q^T B_q, A_q and B_q published 64 x 64 tiles [k][m], [k][n]; c in the accumulator layout: rows
// wr * 16 + 4 v + fq, columns w2 * 32 + 16 j + fr of wavefront (wr, w2).  src.a(q), src.b(q): the tiles; src.ready(q, q1, lane):
// how many steps from q on have both their tiles (one look, wavefront-uniform).
// Where several steps are known to be ready they are pipelined: during the products of a step the next one's tiles go
// from registers to LDS and the loads of the one after the next but one are issued, one or two between any two MFMAs
// (loads and stores in front of the products cost 0.9 us a step: 2.7 us against 1.7 us of matrix time).  The number
// of loads in flight must not depend on a branch, or every wait becomes a wait for all of them.
// LDS: two pairs of tiles, one barrier per step; step number n reads the pair n & 1.
__device__ __forceinline__ void flow_product(const double* As, const double* Bs, int xa, int xb, int kk, d4 (&c)[2])   // rows 8 kk .. 8 kk + 7
{
    const d2 a = pair(As + xa + kk * 512), b = pair(Bs + xb + kk * 512), e = pair(Bs + xb + 32 + kk * 512);
    c[0] = mfma4(a.x, b.x, c[0]);
    c[1] = mfma4(a.x, e.x, c[1]);
    c[0] = mfma4(a.y, b.y, c[0]);
    c[1] = mfma4(a.y, e.y, c[1]);
}

template <class Src>
__device__ __forceinline__ void flow_sum(const FlowP& f, double* lds, const Src& src, int q0, int q1, d4 (&c)[2])
{
    const int lane = here(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
    const int x0 = wave * 512 + 2 * lane;                      // this lane's first pair of a tile: rows wave * 8 + 2 u and the next, column lane
    const int ra = fq * 128 + 2 * (wr * 16 + fr), rb = fq * 128 + 2 * (w2 * 32 + fr);
    auto load = [&](int q, d2 (&pa)[4], d2 (&pb)[4]) {
        const double* a = src.a(q);
        const double* b = src.b(q);
#pragma unroll
        for (int u = 0; u < 4; ++u) { pa[u] = ld_pair(a, x0 + u * 128); pb[u] = ld_pair(b, x0 + u * 128); }
    };
    auto store = [&](double* As, const d2 (&pa)[4], const d2 (&pb)[4]) {
        const int x = here(x0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            pair(As + x + u * 128) = pa[u];
            pair(As + TILE + x + u * 128) = pb[u];
        }
    };
    auto products = [&](const double* As) {
        const int xa = here(ra), xb = here(rb);
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) flow_product(As, As + TILE, xa, xb, kk, c);
    };
    // the products of the pair at As; meanwhile pa, pb to the pair at next and the loads of step q into pa, pb
    auto step = [&](const double* As, double* next, d2 (&pa)[4], d2 (&pb)[4], int q) {
        const int xa = here(ra), xb = here(rb), x = here(x0);
        const double* a = src.a(q);
        const double* b = src.b(q);
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            flow_product(As, As + TILE, xa, xb, kk, c);
            const int u = kk & 3;
            d2 (&pp)[4] = kk < 4 ? pa : pb;
            pair(next + (kk < 4 ? 0 : TILE) + x + u * 128) = pp[u];
            pp[u] = ld_pair(kk < 4 ? a : b, x0 + u * 128);
        }
    };
    d2 pa[4], pb[4], na[4], nb[4];
    double* cur = lds;                   // pair of LDS tiles of the next step, and the other one
    double* alt = lds + 2 * TILE;
    int known = q0;                      // the tiles of the steps before this one are ready
    for (int q = q0; q < q1;) {
        for (FlowPatience w; known <= q;) {                  // wavefront-uniform
            const int k = src.ready(q, q1, lane);
            if (k > 0) known = min(q + k, q1);
            else if (flow_gives_up(f, w)) known = q1;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        if (known - q < 4) {
            load(q, pa, pb);
            store(cur, pa, pb);
            __syncthreads();
            products(cur);
            double* t = cur; cur = alt; alt = t;
            ++q;
            continue;
        }
        const int end = known - 1;
        load(q, pa, pb);
        load(q + 1, na, nb);
        store(cur, pa, pb);
        load(q + 2, pa, pb);
        __syncthreads();
        while (q + 1 < end) {
            step(cur, alt, na, nb, min(q + 3, end));
            __syncthreads();
            step(alt, cur, pa, pb, min(q + 4, end));
            __syncthreads();
            q += 2;
        }
        if (q < end) {
            step(cur, alt, na, nb, end);
            __syncthreads();
            double* t = cur; cur = alt; alt = t;
            ++q;
        }
        products(cur);
        double* t = cur; cur = alt; alt = t;
        ++q;
    }
}

// u = -G c for the finished sum c of a tile in row i of tiles, G = the block inverse of that row (its transpose is
// gt[i]).  u: row tiles {w2, 3 - w2} (G is lower triangular: 20 of 32 (k-step, tile) pairs either way), columns
// wr * 16 ..  steps: how many the sum had (the product takes the pair of LDS tiles that its last step did not read).
template <int W>
__device__ __forceinline__ void flow_tri_product(const double* Gs, const double* Cs, int wr, int fr, int fq, d4 (&u)[2])
{
    const int rc = here(fq * 128 + 2 * (wr * 16 + fr)), r0 = here(fq * 128 + 2 * (W * 16 + fr)), r1 = here(fq * 128 + 2 * ((3 - W) * 16 + fr));
#pragma unroll
    for (int kk = 0; kk < 8 - 2 * W; ++kk) {
        const d2 b = pair(Cs + rc + kk * 512), h = pair(Gs + r1 + kk * 512);
        if (kk < 2 * W + 2) {
            const d2 g = pair(Gs + r0 + kk * 512);
            u[0] = mfma4(g.x, b.x, u[0]);
            u[0] = mfma4(g.y, b.y, u[0]);
        }
        u[1] = mfma4(h.x, b.x, u[1]);
        u[1] = mfma4(h.y, b.y, u[1]);
    }
}

__device__ __forceinline__ void flow_row_product(const FlowP& f, double* lds, int i, int steps, const d4 (&c)[2], d4 (&u)[2])
{
    const int lane = here(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
    double* Gs = lds + (steps & 1) * 2 * TILE;
    double* Cs = Gs + TILE;
    flow_wait(f, tile_word(f, i, i), lane == 0);
    const int x0 = here(wave * 512 + 2 * lane);
    d2 pg[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) pg[x] = ld_pair(f.gt + (int64_t)i * TILE, x0 + x * 128);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) Cs[here(pair_at(wr * 16 + fq, w2 * 32 + 16 * j + fr)) + v * 256] = -c[j][v];
#pragma unroll
    for (int x = 0; x < 4; ++x) pair(Gs + x0 + x * 128) = pg[x];
    __syncthreads();
    u[0] = d4{0.0, 0.0, 0.0, 0.0};
    u[1] = d4{0.0, 0.0, 0.0, 0.0};
    if (w2 == 0) flow_tri_product<0>(Gs, Cs, wr, fr, fq, u);
    else flow_tri_product<1>(Gs, Cs, wr, fr, fq, u);
}

// The last panel, that of row p = k - 2 of tiles, of the sum c for D(k, which) (see Queue1).  Tile (p, k) is wanted here as soon as
// the chain has the block inverse of row p; taking it from the workgroup that owns it would put its publication and another
// look between that inverse and the chain's next block but one.  So its sum is handed over before it meets the inverse
// (sum_tile), and the product with the inverse is formed here too.  tilesN, vec: of the elimination.  steps: as in flow_row_product.
template <bool ELIM>
__device__ __forceinline__ void flow_last_panel(const FlowP& f, const double* tilesN, const double* vec, double* lds, int k, int which, int steps,
                                                d4 (&c)[2])
{
    const int lane = here(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
    const int p = k - 2;
    flow_wait(f, hand_word(f, k, 2), lane == 0);
    d4 s[2], u[2];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const d2 y = ld_pair(sum_tile(f, k), x * 2 * NT + 2 * here(threadIdx.x));
        s[x >> 1][2 * (x & 1)] = y.x;
        s[x >> 1][2 * (x & 1) + 1] = y.y;
    }
    flow_row_product(f, lds, p, steps, s, u);
    double* As = lds + ((steps + 1) & 1) * 2 * TILE;             // (the pair that the last step of the sum has read)
    double* Bs = As + TILE;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int m = (h ? 3 - w2 : w2) * 16 + 4 * v + fq, n = wr * 16 + fr;
            Bs[pair_at(m, n)] = u[h][v];
            if (ELIM && which == 1) As[pair_at(m, n)] = u[h][v] * ld_shared(vec + 2 * NB * p + m);
        }
    if (which == 0) {
        flow_wait(f, tile_word(f, p, p + 1), lane == 0);
        const double* a = ELIM ? tilesN + ((int64_t)p * f.T + p + 1) * TILE : tile_at(f, p, p + 1);
        const int x0 = here(wave * 512 + 2 * lane);
        d2 pa[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) pa[x] = ld_pair(a, x0 + x * 128);
#pragma unroll
        for (int x = 0; x < 4; ++x) pair(As + x0 + x * 128) = pa[x];
    } else if (!ELIM) {
        As = Bs;
    }
    __syncthreads();
    const int xa = here(fq * 128 + 2 * (wr * 16 + fr)), xb = here(fq * 128 + 2 * (w2 * 32 + fr));
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) flow_product(As, Bs, xa, xb, kk, c);
}

// The sum of tile (i, i + 2) before its product with the block inverse of row i, for those who wait for the tile (flow_last_panel);
// every thread finds its own values again.
__device__ __forceinline__ void flow_hand_sum(const FlowP& f, int i, const d4 (&c)[2])
{
#pragma unroll
    for (int x = 0; x < 4; ++x)
        st_pair(sum_tile(f, i + 2), x * 2 * NT + 2 * here(threadIdx.x), d2{c[x >> 1][2 * (x & 1)], c[x >> 1][2 * (x & 1) + 1]});
    flow_publish(hand_word(f, i + 2, 2));
}

// steps q, q + 1, ... whose tiles (q, i) and (q, j) are both published, out of the next 32
__device__ __forceinline__ int ready_pairs(const FlowP& f, int i, int j, int q, int q1, int lane)
{
    const int s = min(q + (lane & 31), q1 - 1);
    const unsigned long long m = __ballot(ld_word(tile_word(f, s, lane < 32 ? i : j)) != 0);
    const unsigned both = (unsigned)m & (unsigned)(m >> 32);
    return both == ~0u ? 32 : __builtin_ctz(~both);
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
    return __builtin_amdgcn_readfirstlane(*slot);
}

// the queue that the workgroup with this role (its place in the order of arrival) serves first: one each, then dealt so that
// however many have arrived, the queues have theirs in proportion (other launches may hold compute units for a while)
__device__ __forceinline__ int flow_serves(const FlowP& f, int role)
{
    if (role <= 3) return role;
    const int all = f.n1 + f.n2 + f.n3;
    if ((role + 1) * f.n1 / all > role * f.n1 / all) return 1;
    const int rest = role - role * f.n1 / all;          // of the others, this one's place among those not on queue 1
    return (rest + 1) * f.n2 / (f.n2 + f.n3) > rest * f.n2 / (f.n2 + f.n3) ? 2 : 3;
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

// minus tile (i, j), i <= j, of H (0 past d) in the accumulator layout, lambda added on the diagonal.  H is read on and below its
// diagonal only (of a diagonal tile the chain uses that part): the mirrored tile, 16 lanes a row apart, each line of 128
// bytes in four loads of the same wavefront.
__device__ __forceinline__ void flow_init_h(const FlowInverseP& p, int i, int j, double lam, d4 (&c)[2])
{
    const int lane = here(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
    const int d = p.f.d;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int gm = NB * i + wr * 16 + 4 * v + fq, gn = NB * j + w2 * 32 + 16 * h + fr;
            double x = (gm < d && gn < d) ? p.H[(int64_t)max(gm, gn) * d + min(gm, gn)] : 0.0;
            if (gm == gn) x += lam;
            c[h][v] = -x;
        }
}

struct SumR {      // R_qi^T R_qj; X_qi^T X_qj; R_qi^T X_qj
    FlowP f; int i, j;
    __device__ const double* a(int q) const { return tile_at(f, q, i); }
    __device__ const double* b(int q) const { return tile_at(f, q, j); }
    __device__ int ready(int q, int q1, int lane) const { return ready_pairs(f, i, j, q, q1, lane); }
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
// What a block takes, in us (256 x 2304, inverse / elimination, 12.5 / 13.3 in all): waiting for the sums 0.4, product with the
// inverse 0.6, tile to LDS and memory 1.0 / 1.3, product off the diagonal block 1.0, that to LDS 0.3, the block 7.4, loads and stores
// of its results 1.2 / 1.7, their way to memory 0.5.  (15.3 with 8-byte exchange, an L2 write-back per word, and the sums behind
// tile (k - 2, k)'s own publication.)
__device__ __forceinline__ void chain_tiles(int wave, int (&rt)[2], int (&ct)[2])
{
    rt[0] = wave < 4 ? wave : wave == 4 ? 1 : wave == 6 ? 3 : 2;
    ct[0] = wave < 4 ? 0 : wave == 7 ? 2 : 1;
    rt[1] = 3;
    ct[1] = wave == 1 ? 2 : 3;
}

// The block inverse G (lower triangular, DL-strided in LDS) as A operand of the row tiles {W, 3 - W}: row tile t needs the
// k-steps 0 .. 4 t + 3 only, 20 of 32 (k-step, tile) pairs for either W, two k-steps (rows 8 kk + 2 fq and the next) at a time:
// g[0 .. 2 W + 1] are tile W's, the rest 3 - W's.
template <int W>
__device__ __forceinline__ void chain_load_inverse(const double* Xm, int fr, int fq, d2 (&g)[10])
{
    const int r0 = here((W * 16 + fr) * DL + 2 * fq), r1 = here(((3 - W) * 16 + fr) * DL + 2 * fq);
#pragma unroll
    for (int x = 0; x < 10; ++x) {
        const bool lo = x < 2 * W + 2;
        g[x] = pair(Xm + (lo ? r0 : r1) + 8 * (lo ? x : x - 2 * W - 2));
    }
}

template <int W>
__device__ __forceinline__ void chain_row_product(const d2 (&g)[10], const d2 (&vb)[8], d4 (&u)[2])
{
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        if (kk < 2 * W + 2) u[0] = mfma4(g[kk].x, vb[kk].x, u[0]);
        if (kk < 8 - 2 * W) u[1] = mfma4(g[2 * W + 2 + kk].x, vb[kk].x, u[1]);
        if (kk < 2 * W + 2) u[0] = mfma4(g[kk].y, vb[kk].y, u[0]);
        if (kk < 8 - 2 * W) u[1] = mfma4(g[2 * W + 2 + kk].y, vb[kk].y, u[1]);
    }
}

// ELIM: the elimination (tiles U, tilesN = Un = U / pivot, vec: see FlowElimP), else the Cholesky factorization (tiles R above and
// X on the diagonal).  first(m, n): element (m, n) of diagonal block 0.
template <bool ELIM, class First>
__device__ __forceinline__ void flow_chain(const FlowP& f, double* tilesN, double* vec, double* lds, First first)
{
    double* Am = lds + SWEEP_LDS;
    double* Xm = Am + NB * DL;
    double* Vs = Xm + NB * DL;                   // tile (k - 1, k) of U or R, and (ELIM) of Un
    double* Vn = ELIM ? Vs + TILE : Vs;
    d4 c[2];
    d2 vb[8], g[10];
    // chol_block writes the lower triangle of the inverse, whole 16 x 16 tiles on the diagonal included (zeros above it);
    // the tiles above stay as they are.  (Past d the last block's inverse is the identity: its rows meet zeros only.)
    for (int x = threadIdx.x; x < NB * NB; x += NT) Xm[(x >> 6) * DL + (x & 63)] = 0.0;
    // The word of a block inverse: whichever wavefront is the last to know its stores done sets it (a count in LDS), so that
    // none waits for another's before it goes on.  (Its own it does wait for here: with the word put off behind the next
    // product, 2 us later, the chain is that much shorter, but the sums it needs come later too, 1036 against 1071 us for a
    // layer of 1000 x 2048.)
    int* stored = reinterpret_cast<int*>(lds + SWEEP_LDS) - 1;
    if (threadIdx.x == 0) *stored = 0;
    auto publish_inverse = [&](int k) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
        if ((threadIdx.x & 63) == 0 && __hip_atomic_fetch_add(stored, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == (NT / 64) * (k + 1) - 1) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            st_word(tile_word(f, k, k), 1);
        }
    };
    bool have = false;                           // the sums of the next block are loaded
    for (int k = 0; k < f.T; ++k) {
        const int nb = min(NB, f.d - NB * k);
        const int tid = here(threadIdx.x), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
        int rt[2], ct[2];
        chain_tiles(wave, rt, ct);
        if (ELIM) {                                  // elim_block reads the upper triangle, chol_block the lower one
            const int a0 = rt[0], a1 = rt[1];
            rt[0] = ct[0]; rt[1] = ct[1];
            ct[0] = a0; ct[1] = a1;
        }
        const bool second = wave == 1 || wave == 2;
        const int t[2] = {w2, 3 - w2};               // row tiles of the product with the block inverse
        auto load_sums = [&](int k) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            const double* D = tile_at(f, k, k);
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) vb[kk] = ld_pair(hand_tile(f, k), (4 * kk + fq) * 128 + 2 * (wr * 16 + fr));
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (h == 0 || second) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) c[h][v] = ld_shared(D + pair_at(rt[h] * 16 + 4 * v + fq, ct[h] * 16 + fr));
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
        auto diag_product = [&](int h) {             // c[h] -= (tile (k - 1, k) of R or Un)[:, row tile]^T (of R or U)[:, column tile]
            const int ra = here(swz(fq, rt[h] * 16 + fr)), rb = here(swz(fq, ct[h] * 16 + fr));
#pragma unroll
            for (int ks = 0; ks < 16; ++ks) c[h] = mfma4(-Vn[ra + ks * 256], Vs[rb + ks * 256], c[h]);
        };
        if (k == 0) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (h == 0 || second) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int m = rt[h] * 16 + 4 * v + fq, n = ct[h] * 16 + fr;
                        c[h][v] = (m < nb && n < nb) ? first(m, n) : 0.0;
                    }
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
            double* Rn = tilesN + ((int64_t)(k - 1) * f.T + k) * TILE;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int n = wr * 16 + fr, at = here(swz(t[i] * 16 + fq, n));
                d4 un;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    Vs[at + v * 256] = u[i][v];
                    if (ELIM) {
                        un[v] = u[i][v] * lds[t[i] * 16 + 4 * v + fq];      // 1 / pivot of the block before
                        Vn[at + v * 256] = un[v];
                    }
                }
                st_rows(R, t[i] * 16, n, fq, u[i]);
                if (ELIM) st_rows(Rn, t[i] * 16, n, fq, un);
            }
            __syncthreads();
            diag_product(0);
            __builtin_amdgcn_s_waitcnt(0);
        }
        store_diag(0, nb);
        __syncthreads();
        if (k > 0 && tid == NT - 64) {           // a wavefront that the sweeps leave idle
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            st_word(tile_word(f, k - 1, k), 1);
        }
        int seen = 1;                            // words of the next block's sums, looked at while the last sweep runs
        auto beside = [&]() {
            if (second) {
                if (k > 0) diag_product(1);
                store_diag(1, nb);
            }
        };
        auto ahead = [&]() {
            if (lane < 2 && k + 1 < f.T) seen = ld_word(hand_word(f, k + 1, lane));
        };
        if constexpr (ELIM) elim_block(Am, Xm, lds, f.notpd, beside, ahead);
        else chol_block(Am, Xm, lds, f.notpd, beside, ahead);
        // the next block's sums: looked for before and after the stores of the block inverse
        have = k + 1 < f.T && __all(seen != 0);
        if (have) load_sums(k + 1);
        double* Gt = f.gt + (int64_t)k * TILE;
        double* G = tile_at(f, k, k);
        double* Gn = tilesN + ((int64_t)k * f.T + k) * TILE;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int y = wave * 8 + 2 * x, at = y * 64 + 2 * lane;
            st_pair(Gt, at, pair(Xm + lane * DL + y));
            if (ELIM) st_pair(Gn, at, d2{y < lane ? Am[y * DL + lane] * lds[y] : 0.0, y + 1 < lane ? Am[(y + 1) * DL + lane] * lds[y + 1] : 0.0});
            else st_pair(G, at, d2{Xm[y * DL + lane], Xm[(y + 1) * DL + lane]});
        }
        if (ELIM && wave == 0) {
            st_shared(vec + 2 * NB * k + lane, lds[lane]);
            st_shared(vec + 2 * NB * k + NB + lane, 0.5 / Am[lane * DL + lane]);
        }
        if (k + 1 < f.T) {
            if (!have) {
                have = __all(lane < 2 ? ld_word(hand_word(f, k + 1, lane)) != 0 : true);
                if (have) load_sums(k + 1);
            }
            if (w2 == 0) chain_load_inverse<0>(Xm, fr, fq, g);
            else chain_load_inverse<1>(Xm, fr, fq, g);
        }
        publish_inverse(k);
    }
}

__device__ __forceinline__ void flow_inverse(const FlowInverseP& p, double* lds, int& slot)
{
    const FlowP& f = p.f;
    const int T = f.T;
    double* tiles = lds + SWEEP_LDS;
    const int role = flow_ticket(f, FW_ROLE, &slot);
    if (role == 0) {
        const double lam = flow_lambda(p, tiles);
        flow_chain<false>(f, nullptr, nullptr, lds, [&](int m, int n) { return p.H[(int64_t)max(m, n) * f.d + min(m, n)] + (m == n ? lam : 0.0); });
    } else if (flow_serves(f, role) == 1) {
        Queue1 q1;
        const int n = queue1_length(T);
        for (;;) {
            const int t = flow_ticket(f, FW_QUEUE1, &slot);
            if (t >= n) break;
            const Queue1Item it = q1.at(t, T);
            const int lane = here(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
            const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
            d4 c[2], u[2];
            if (it.kind == 0) {
                flow_init_h(p, it.i, it.j, 0.0, c);
                flow_sum(f, tiles, SumR{f, it.i, it.j}, 0, it.i, c);
                if (it.j == it.i + 2) flow_hand_sum(f, it.i, c);
                flow_row_product(f, tiles, it.i, it.i, c, u);
                double* out = tile_at(f, it.i, it.j);
#pragma unroll
                for (int h = 0; h < 2; ++h) st_rows(out, (h ? 3 - w2 : w2) * 16, wr * 16 + fr, fq, u[h]);
                flow_publish(tile_word(f, it.i, it.j));
            } else {
                const int k = it.i, ti = it.j ? k : k - 1;
                const double lam = it.j ? flow_lambda(p, tiles) : 0.0;
                flow_init_h(p, ti, k, lam, c);
                flow_sum(f, tiles, SumR{f, ti, k}, 0, k - 2, c);
                if (k > 1) flow_last_panel<false>(f, nullptr, nullptr, tiles, k, it.j, k - 2, c);
                double* out = it.j ? tile_at(f, k, k) : hand_tile(f, k);
#pragma unroll
                for (int h = 0; h < 2; ++h) st_rows(out, wr * 16, w2 * 32 + 16 * h + fr, fq, -c[h]);
                flow_publish(hand_word(f, k, it.j));
            }
        }
    }
    const int nx = T * (T - 1) / 2, nh = T * (T + 1) / 2;      // (whoever does not serve queue 1 first serves queue 2)
    for (;;) {
        const int t = flow_ticket(f, FW_QUEUE2, &slot);
        if (t >= nx + nh) break;
        const int lane = here(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
        d4 c[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}}, u[2];
        if (t < nx) {
            int i, j;
            tri_decode(t, i, j);
            ++i;
            flow_sum(f, tiles, SumR{f, i, j}, j, i, c);          // tile (q, j), q >= j, is X_qj
            flow_row_product(f, tiles, i, i - j, c, u);
            double* out = tile_at(f, i, j);
#pragma unroll
            for (int h = 0; h < 2; ++h) st_rows(out, (h ? 3 - w2 : w2) * 16, wr * 16 + fr, fq, u[h]);
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
                    if (gm < f.d && gn < f.d) p.Hinv[(int64_t)gm * f.d + gn] = c[h][v];
                }
        }
    }
    if (threadIdx.x == 0 && ld_word(f.words + FW_ABORT) != 0) *f.stalled = 1;
}

__global__ __launch_bounds__(NT, 2) void flow_inverse_kernel(FlowInverseP p)
{
    __shared__ __attribute__((aligned(16))) double lds[FLOW_LDS];
    __shared__ int slot;
    flow_inverse(p, lds, slot);
}

// Several layers in one launch: the b-th workgroup to arrive works on layer layer_of[b].  A layer's entries are consecutive
// and the number is drawn, not the workgroup's index, so the workgroups that wait are never those of a layer whose others
// cannot become resident.
__device__ __forceinline__ int batch_layer(int* arrivals, const uint16_t* layer_of, int& slot)
{
    if (threadIdx.x == 0) slot = layer_of[min(atomicAdd(arrivals, 1), (int)gridDim.x - 1)];
    __syncthreads();
    const int l = __builtin_amdgcn_readfirstlane(slot);
    __syncthreads();
    return l;
}

__global__ __launch_bounds__(NT, 2) void flow_inverse_batch_kernel(const FlowInverseP* __restrict__ layers, const uint16_t* __restrict__ layer_of,
                                                                   int* __restrict__ arrivals)
{
    __shared__ __attribute__((aligned(16))) double lds[FLOW_LDS];
    __shared__ int slot;
    const FlowInverseP p = layers[batch_layer(arrivals, layer_of, slot)];
    flow_inverse(p, lds, slot);
}

// ---------------------------------------------------------------------------
// The shared-Hinv elimination (Eq. 12) and the column loop (Section 4.2 steps 4-5) in one launch.  With A = Hinv in
// processing order (gathered through perm when a tile is started):
//   U_ij = G_i (A_ij - sum_{q < i} Un_qi^T U_qj), i < j, Un = D^-1 U;  G_i, the pivots and Un_ii from elim_block   (queue 1)
// and for the rows of W, which do not interact, in groups g of 64 rows and parts s of RS rows:
//   W(p, g) = W[:, block p] (gathered, widened) - sum_{q < p - 1} D_qg^T Un_qp                                       (queue 3)
//   C(p, s): the 64 sequential steps of block p for its rows, on W(p, g) less the share of block p - 1 that C(p - 1, s)
//            computed; leaves D_p (w - q, [column][row]), the codes, the loss terms, and its share for block p + 1.  (queue 2)
// RS = 8 NR: NR rows per wavefront (see column_rows).  Queues 2 and 3 go through the blocks for NGC groups of rows at a time (see
// group_run), the last run the rest.
struct FlowElimP {
    FlowP f;
    double* tilesN;        // T x T: Un; on the diagonal Un inside the block (0 on and below its diagonal)
    double* vec;           // T x 128: reciprocal pivots, 1 / (2 pivot)
    const double* Hu;      // Hinv (original order, upper triangle)
    const int* perm;
    const float* W; int R, G, gs, NG, NGC;
    const double* scale; const double* zero; double maxq;
    uint8_t* codesT; int Rp; double* lossrow;
    double* Wout;          // R x d, processing order, or null
    double* wt;            // T x NG tiles: W(p, g), [row][column]
    double* dt;            // T x NG tiles: D, [column][row]
    double* corr;          // 2 x Rp x 64: the share of the block before, by parity of the block
};

__device__ __forceinline__ int* group_word(const FlowElimP& p, int blk, int g) { return p.f.words + FW_HEAD + p.f.T * p.f.T + 3 * p.f.T + blk * p.NG + g; }
__device__ __forceinline__ int* part_word(const FlowElimP& p, int blk, int s, int parts) { return p.f.words + FW_HEAD + p.f.T * p.f.T + 3 * p.f.T + p.f.T * p.NG + blk * parts + s; }

struct SumU {      // Un_qi^T U_qj
    FlowP f; const double* tilesN; int i, j;
    __device__ const double* a(int q) const { return tilesN + ((int64_t)q * f.T + i) * TILE; }
    __device__ const double* b(int q) const { return tile_at(f, q, j); }
    __device__ int ready(int q, int q1, int lane) const { return ready_pairs(f, i, j, q, q1, lane); }
};

template <int PER>
struct SumW {      // D_qg^T Un_qp; a step is ready when all PER parts of the group and the tile (q, p) are
    const FlowElimP& e; int p, g;
    __device__ const double* a(int q) const { return e.dt + ((int64_t)q * e.NG + g) * TILE; }
    __device__ const double* b(int q) const { return e.tilesN + ((int64_t)q * e.f.T + p) * TILE; }
    __device__ int ready(int q, int q1, int lane) const
    {
        constexpr int M = PER + 1, STEPS = 64 / M;
        const int n = min(STEPS, q1 - q), st = lane / M, x = lane % M;
        int v = 1;
        if (st < n) v = ld_word(x < PER ? part_word(e, q + st, g * PER + x, e.NG * PER) : tile_word(e.f, q + st, p));
        const unsigned long long m = __ballot(v != 0);
        int k = 0;
        while (k < n && ((m >> (k * M)) & ((1ull << M) - 1)) == (1ull << M) - 1) ++k;
        return k;
    }
};

// element (m, n) of A = Hinv in processing order; flow_init_a: minus tile (i, j) of A (0 past d) in the accumulator layout
__device__ __forceinline__ double flow_hinv(const FlowElimP& p, int m, int n)
{
    const int d = p.f.d;
    const int pm = min(max(p.perm[m], 0), d - 1), pn = min(max(p.perm[n], 0), d - 1);
    return p.Hu[(int64_t)min(pm, pn) * d + max(pm, pn)];
}

__device__ __forceinline__ void flow_init_a(const FlowElimP& p, int i, int j, d4 (&c)[2])
{
    const int lane = here(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int gm = NB * i + wr * 16 + 4 * v + fq, gn = NB * j + w2 * 32 + 16 * h + fr;
            c[h][v] = (gm < p.f.d && gn < p.f.d) ? -flow_hinv(p, gm, gn) : 0.0;
        }
}

// C(blk, s) by one workgroup; lds: two tiles, D and the codes of its rows
template <int NR>
__device__ __forceinline__ void flow_columns(const FlowElimP& p, double* lds, int blk, int s)
{
    constexpr int RS = 8 * NR, PER = 64 / RS;
    const FlowP& f = p.f;
    const int tid = here(threadIdx.x), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int d = f.d, o = NB * blk, nb = min(NB, d - o), parts = p.NG * PER;
    const int g = s / PER, r0 = (s % PER) * RS + wave * NR;      // first row of this wavefront inside the group
    const bool more = blk + 1 < f.T;
    double* Us = lds;
    double* Vs = Us + TILE;
    double* Ds = Vs + TILE;                                      // [column][RS]
    uint8_t* Cs = reinterpret_cast<uint8_t*>(Ds + NB * RS);      // [column][RS]
    double ws[NR], w0[NR], sc[NR], ze[NR];
    const int col = min(o + lane, d - 1);
    const int gcol = min(max(p.perm[col], 0), d - 1) / p.gs;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int64_t gi = (int64_t)min(NB * g + r0 + r, p.R - 1) * p.G + gcol;
        sc[r] = p.scale[gi];
        ze[r] = p.zero[gi];
    }
    flow_wait(f, lane == 0 ? tile_word(f, blk, blk) : lane == 1 ? group_word(p, blk, g) : part_word(p, max(blk, 1) - 1, s, parts),
              lane < (blk > 0 ? 3 : 2));
    {
        d2 un[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) un[x] = ld_pair(p.tilesN + ((int64_t)blk * f.T + blk) * TILE, wave * 512 + x * 128 + 2 * lane);
        const double* wt = p.wt + ((int64_t)blk * p.NG + g) * TILE + r0 * 64 + lane;
        const double* cin = p.corr + ((int64_t)(blk & 1) * p.NG * NB + NB * g + r0) * 64 + lane;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            w0[r] = ld_shared(wt + r * 64);
            if (blk > 0) w0[r] -= ld_shared(cin + r * 64);
        }
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            Us[wave * 512 + x * 128 + lane] = un[x].x;
            Us[wave * 512 + x * 128 + 64 + lane] = un[x].y;
        }
    }
    const double hp = ld_shared(p.vec + 2 * NB * blk + NB + lane);
    __syncthreads();
    double mycode[NR], mydiff[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) { ws[r] = w0[r]; mycode[r] = 0.0; mydiff[r] = 0.0; }
    // what comes after the steps and is there already: the pivot rows above the next block's columns, the loss so far
    bool ahead = more && __all(lane == 0 ? ld_word(tile_word(f, blk, blk + 1)) != 0 : true);
    d2 t[4];
    auto load_next = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll
        for (int x = 0; x < 4; ++x) t[x] = ld_pair(p.tilesN + ((int64_t)blk * f.T + blk + 1) * TILE, wave * 512 + x * 128 + 2 * lane);
    };
    if (ahead) load_next();
    double loss_before[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) loss_before[r] = ld_shared(p.lossrow + min(NB * g + r0 + r, p.R - 1));
    bool suspect = false;
    chain_steps<false, NR, NB>(ws, Us, sc, ze, p.maxq, nb, lane, mycode, mydiff, suspect);
    if (__any(suspect)) {                    // wavefront-uniform; practically never taken
#pragma unroll
        for (int r = 0; r < NR; ++r) ws[r] = w0[r];
        chain_steps<true, NR, NB>(ws, Us, sc, ze, p.maxq, nb, lane, mycode, mydiff, suspect);
    }
    if (more) {
        if (!ahead) {
            flow_wait(f, tile_word(f, blk, blk + 1), lane == 0);
            load_next();
        }
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            Vs[wave * 512 + x * 128 + lane] = t[x].x;
            Vs[wave * 512 + x * 128 + 64 + lane] = t[x].y;
        }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        if (lane >= nb) { mydiff[r] = 0.0; mycode[r] = 0.0; }
        Ds[lane * RS + wave * NR + r] = mydiff[r];
        Cs[lane * RS + wave * NR + r] = (uint8_t)mycode[r];
    }
    __syncthreads();
    if (more) {
        // the share of the next block's columns, rows of D times a 64 x 64 tile: of 32 rows as one 16 x 16 tile a wavefront on the
        // matrix cores (with 16 rows half the wavefronts have one and wait for 16 dependent products: 983 -> 998 us for
        // 1000 x 2048), of fewer as the steps went.  20 layers of up to 1024 rows in one call 363 -> 348 us.
        double* cout = p.corr + ((int64_t)((blk + 1) & 1) * p.NG * NB + NB * g + (s % PER) * RS) * 64;
        if constexpr (NR == 4) {
            const int fr = lane & 15, fq = lane >> 4, m0 = (wave >> 2) * 16, n0 = (wave & 3) * 16;
            const int ra = here(fq * RS + m0 + fr), rb = here(fq * 64 + n0 + fr);
            d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int ks = 0; ks < 16; ++ks) acc = mfma4(Ds[ra + ks * 4 * RS], Vs[rb + ks * 256], acc);
#pragma unroll
            for (int v = 0; v < 4; ++v) st_shared(cout + (m0 + 4 * v + fq) * 64 + n0 + fr, acc[v]);
        } else {
            double acc[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[r] = 0.0;
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const double v = Vs[k * 64 + lane];
#pragma unroll
                for (int r = 0; r < NR; ++r) acc[r] = fma(chain_readlane(mydiff[r], k), v, acc[r]);
            }
#pragma unroll
            for (int r = 0; r < NR; ++r) st_shared(cout + (wave * NR + r) * 64 + lane, acc[r]);
        }
        if (blk + 2 < f.T) {
            double* dt = p.dt + ((int64_t)blk * p.NG + g) * TILE;
#pragma unroll
            for (int x = 0; x < (NR + 1) / 2; ++x) {
                const int e = tid + NT * x, c2 = e / RS, r = e % RS;      // columns 2 c2 and 2 c2 + 1 of row r
                if (c2 < NB / 2) st_pair(dt, c2 * 128 + 2 * ((s % PER) * RS + r), d2{Ds[2 * c2 * RS + r], Ds[(2 * c2 + 1) * RS + r]});
            }
        }
    }
    // the codes, 8 rows at a time (codesT is padded to whole groups of rows)
    if (tid < NB * NR && tid / NR < nb)
        *reinterpret_cast<unsigned long long*>(p.codesT + (int64_t)(o + tid / NR) * p.Rp + NB * g + (s % PER) * RS + 8 * (tid % NR)) =
            reinterpret_cast<const unsigned long long*>(Cs)[tid];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int row = NB * g + r0 + r;
        double loss = mydiff[r] * mydiff[r] * hp;
        if (lane >= nb) loss = 0.0;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) loss += __shfl_xor(loss, off);
        if (row < p.R) {
            if (lane == 0) st_shared(p.lossrow + row, loss_before[r] + loss);
            if (p.Wout && lane < nb) p.Wout[(int64_t)row * d + o + lane] = ws[r];
        }
    }
    flow_publish(part_word(p, blk, s, parts));
}

// Ticket t of queue 2 (per = 64 / RS parts to a group) or 3 (per = 1): block and part / group.
__device__ __forceinline__ void flow_rows_item(const FlowElimP& p, int t, int per, int& blk, int& x)
{
    int n = p.NG * per, x0 = 0;
    if (p.NGC < p.NG) {
        const int run = t / (p.f.T * p.NGC * per);
        x0 = run * p.NGC * per;
        n = min(p.NGC * per, n - x0);
        t -= p.f.T * x0;
    }
    blk = t / n;
    x = x0 + t - blk * n;
}

template <int NR>
__device__ __forceinline__ void flow_eliminate(const FlowElimP& p, double* lds, int& slot)
{
    constexpr int PER = 64 / (8 * NR);
    const FlowP& f = p.f;
    const int T = f.T;
    double* tiles = lds + SWEEP_LDS;
    const int role = flow_ticket(f, FW_ROLE, &slot);
    if (role == 0) flow_chain<true>(f, p.tilesN, p.vec, lds, [&](int m, int n) { return flow_hinv(p, m, n); });
    else if (flow_serves(f, role) == 1) {
        Queue1 q1;
        const int n = queue1_length(T);
        for (;;) {
            const int t = flow_ticket(f, FW_QUEUE1, &slot);
            if (t >= n) break;
            const Queue1Item it = q1.at(t, T);
            const int lane = here(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
            const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
            d4 c[2], u[2];
            if (it.kind == 0) {
                flow_init_a(p, it.i, it.j, c);
                flow_sum(f, tiles, SumU{f, p.tilesN, it.i, it.j}, 0, it.i, c);
                if (it.j == it.i + 2) flow_hand_sum(f, it.i, c);
                flow_row_product(f, tiles, it.i, it.i, c, u);
                double* outn = p.tilesN + ((int64_t)it.i * T + it.j) * TILE;
                const double* rv = p.vec + 2 * NB * it.i;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int m0 = (h ? 3 - w2 : w2) * 16;
                    d4 un;
#pragma unroll
                    for (int v = 0; v < 4; ++v) un[v] = u[h][v] * ld_shared(rv + m0 + 4 * v + fq);
                    st_rows(tile_at(f, it.i, it.j), m0, wr * 16 + fr, fq, u[h]);
                    st_rows(outn, m0, wr * 16 + fr, fq, un);
                }
                flow_publish(tile_word(f, it.i, it.j));
            } else {
                const int k = it.i, ti = it.j ? k : k - 1;
                flow_init_a(p, ti, k, c);
                flow_sum(f, tiles, SumU{f, p.tilesN, ti, k}, 0, k - 2, c);
                if (k > 1) flow_last_panel<true>(f, p.tilesN, p.vec, tiles, k, it.j, k - 2, c);
                double* out = it.j ? tile_at(f, k, k) : hand_tile(f, k);
#pragma unroll
                for (int h = 0; h < 2; ++h) st_rows(out, wr * 16, w2 * 32 + 16 * h + fr, fq, -c[h]);
                flow_publish(hand_word(f, k, it.j));
            }
        }
    }
    // a workgroup whose own queue is empty helps with the others
    for (int turn = 0; turn < 2; ++turn) {
        if ((flow_serves(f, role) == 3) == (turn == 0)) {
            for (;;) {
                const int t = flow_ticket(f, FW_QUEUE3, &slot);
                if (t >= T * p.NG) break;
                int blk, x;
                flow_rows_item(p, t, 1, blk, x);
                const int lane = here(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
                const int wr = wave >> 1, w2 = wave & 1, fr = lane & 15, fq = lane >> 4;
                d4 c[2];
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int gm = NB * x + wr * 16 + 4 * v + fq, gn = NB * blk + w2 * 32 + 16 * h + fr;
                        c[h][v] = (gm < p.R && gn < f.d) ? -(double)p.W[(int64_t)gm * f.d + min(max(p.perm[gn], 0), f.d - 1)] : 0.0;
                    }
                flow_sum(f, tiles, SumW<PER>{p, blk, x}, 0, blk - 1, c);
                double* out = p.wt + ((int64_t)blk * p.NG + x) * TILE;
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int v = 0; v < 4; ++v) st_shared(out + (wr * 16 + 4 * v + fq) * 64 + w2 * 32 + 16 * h + fr, -c[h][v]);
                flow_publish(group_word(p, blk, x));
            }
        } else {
            const int parts = p.NG * PER;
            for (;;) {
                const int t = flow_ticket(f, FW_QUEUE2, &slot);
                if (t >= T * parts) break;
                int blk, x;
                flow_rows_item(p, t, PER, blk, x);
                flow_columns<NR>(p, tiles, blk, x);
            }
        }
    }
    if (threadIdx.x == 0 && ld_word(f.words + FW_ABORT) != 0) *f.stalled = 1;
}

template <int NR>
__global__ __launch_bounds__(NT, 2) void flow_eliminate_kernel(FlowElimP p)
{
    __shared__ __attribute__((aligned(16))) double lds[FLOW_LDS];
    __shared__ int slot;
    flow_eliminate<NR>(p, lds, slot);
}

template <int NR>
__global__ __launch_bounds__(NT, 2) void flow_eliminate_batch_kernel(const FlowElimP* __restrict__ layers, const uint16_t* __restrict__ layer_of,
                                                                     int* __restrict__ arrivals)
{
    __shared__ __attribute__((aligned(16))) double lds[FLOW_LDS];
    __shared__ int slot;
    const FlowElimP p = layers[batch_layer(arrivals, layer_of, slot)];
    flow_eliminate<NR>(p, lds, slot);
}

int64_t flow_inverse_words(int d) { return flow_words((d + NB - 1) / NB); }
// The weights of a part of columns with 1, 2 or 4 rows per wavefront and of a diagonal block in the rules below, in us as they were when the
// lines were drawn.  Now a part takes 7.2 to 8.0, 10.1 to 11.4 and 14.1 to 15.7, a block 12.5 to 13.3.  With those in their place 22 of 306
// shapes (16 .. 65535 rows, 64 .. 8192 columns) would take more rows; of 17 of them measured none gains and most lose (layer, now /
// so: 512 x 3072 1494 / 1565 us, 1000 x 1792 804 / 824, 2048 x 1280 618 / 686, 3000 x 512 315 / 335), so the weights stay.
static const double PART_US[3] = {7.5, 11.0, 18.0}, BLOCK_US = 15.3;
// Rows per wavefront of a part of columns (1, 2 or 4).  A part takes its own time, on top of which its successor
// waits about 2.5 us for it: with few rows the part's time is on a second chain beside the chain of the diagonal blocks, with many the
// workgroups are all busy and what counts is the time per row.  Twice the pure work over all
// workgroups against the chains; measured at 1 / 2 / 4 rows, elimination and columns: 256 x 2304 0.48 / 0.48 / 0.57 ms,
// 2048 x 512 0.140 / 0.140 / 0.157, 1000 x 2048 0.45 / 0.47 / 0.54, 2048 x 1500 0.45 / 0.40 / 0.43, 1024 x 4608 1.99 / 1.70 / 1.63, 8192 x 256
// 0.21 / 0.15 / 0.13; 300 x 4608 1.31 / 1.35 / 1.37, where the rule takes 4.
static int column_rows(int cus, int64_t R, int64_t T)
{
    const double NG = (double)((R + NB - 1) / NB), t = (double)T, products = 2.4 * (t * t * t / 6.0 + NG * t * t / 2.0);
    int best = 1;
    double least = 0.0;
    for (int i = 0; i < 3; ++i) {
        const int nr = 1 << i;
        const double chains = t * std::max(BLOCK_US, PART_US[i] + 2.5), work = 2.0 / (cus - 1) * (products + t * NG * (8 / nr) * PART_US[i]);
        const double time = std::max(chains, work);
        if (i == 0 || time < least) { least = time; best = nr; }
    }
    return best;
}
int64_t flow_eliminate_words(int cus, int d, int R)
{
    const int64_t T = (d + NB - 1) / NB, NG = (R + NB - 1) / NB;
    return flow_words((int)T) + T * NG * (1 + 8 / column_rows(cus, R, T));
}
int64_t flow_eliminate_words_most(int d, int R)
{
    const int64_t T = (d + NB - 1) / NB, NG = (R + NB - 1) / NB;
    return flow_words((int)T) + T * NG * 9;
}
size_t flow_tiles_bytes(int d) { const size_t T = (d + NB - 1) / NB; return T * T * TILE * sizeof(double); }
size_t flow_gt_bytes(int d) { const size_t T = (d + NB - 1) / NB; return 3 * T * TILE * sizeof(double); }
size_t flow_rows_bytes(int d, int R) { const size_t T = (d + NB - 1) / NB, NG = (R + NB - 1) / NB; return T * NG * TILE * sizeof(double); }

// One workgroup per compute unit at most (its LDS), no more than there are tiles to start with.
static int flow_grid(int cus, int64_t tasks) { return (int)(1 + tasks < cus ? 1 + tasks : cus); }

static FlowInverseP inverse_params(const double* H, int d, double damp, double damp_abs, double* Hinv, double* tiles, double* gt, int* words,
                                   int* notpd, int* stalled, int looks, int wgs)
{
    FlowInverseP p;
    p.f.looks = looks;
    p.f.d = d;
    p.f.T = (d + NB - 1) / NB;
    // Two rows of tiles and a half in flight keep the chain fed: with 1.5, 2, 2.5, 3 and 4 the inverse of 4 to 24 blocks of columns takes the
    // same (77, 127, 182, 231, 339 us for 4, 8, 12, 16, 24), that of 36 594, 542, 534, 535, 535, of 48 972, 855, 800, 787, 790, of
    // 64 1732, 1524, 1430, 1407, 1408.  Where the products bound the launch, queue 1 feeds queue 2 and its workgroups go over to that
    // when it is empty, so it has most of them: with 1/2, 3/5, 7/10 and 4/5 of the workgroups 64 blocks 1522, 1447, 1409, 1401 us, 72 2098,
    // 2003, 1921, 1891, 96 4840, 4513, 4323, 4240, 128 11500, 10752, 10182, 9910.
    p.f.n1 = std::max(1, std::min(5 * p.f.T / 2, wgs * 7 / 10));
    p.f.n2 = std::max(1, wgs - 1 - p.f.n1);          // the others: queue 2 (there is no third)
    p.f.n3 = 0;
    p.f.words = words; p.f.tiles = tiles; p.f.gt = gt; p.f.notpd = notpd; p.f.stalled = stalled;
    p.H = H; p.damp = damp; p.damp_abs = damp_abs; p.Hinv = Hinv;
    return p;
}

// Groups of 64 rows that go through all blocks together: rows do not interact, and what a run of them keeps for its later
// blocks (W and D, 64 KB a block and group) should stay in the 256 MB cache on the memory's side; at least 64 groups, which
// keep the workgroups busy, and runs of equal length.  The layer in one run and in runs by this rule: 65535 x 512 3.33 and 3.05 ms
// (2 runs), 65535 x 1024 7.55 and 6.20 (4), 65535 x 2048 19.3 and 16.9 (8), 30000 x 4608 33.2 and 30.4 (9); more runs
// than that lose: 32000 x 512 1.47 in one, 1.55 in two.
static int group_run(int64_t T, int64_t NG)
{
    const int64_t most = std::max<int64_t>(64, (256 << 20) / (64 << 10) / T), runs = (NG + most - 1) / most;
    return (int)((NG + runs - 1) / runs);
}

static FlowElimP eliminate_params(const FlowElimArgs& a)     // all but the numbers of workgroups
{
    FlowElimP p;
    p.f.looks = a.looks;
    p.f.d = a.d;
    p.f.T = (a.d + NB - 1) / NB;
    p.f.words = a.words; p.f.tiles = a.tiles; p.f.gt = a.gt; p.f.notpd = a.notpd; p.f.stalled = a.stalled;
    p.R = a.R; p.G = a.G; p.gs = a.gs; p.NG = (a.R + NB - 1) / NB; p.NGC = group_run(p.f.T, p.NG);
    p.tilesN = a.tilesN; p.vec = a.vec; p.Hu = a.Hinv; p.perm = a.perm; p.W = a.W; p.scale = a.scale; p.zero = a.zero;
    p.maxq = (double)((1 << a.bits) - 1);
    p.codesT = a.codesT; p.Rp = a.Rp; p.lossrow = a.lossrow; p.Wout = a.Wout; p.wt = a.wt; p.dt = a.dt; p.corr = a.corr;
    return p;
}

hipError_t launch_flow_inverse(hipStream_t s, int cus, const double* H, int d, double damp, double damp_abs, double* Hinv, double* tiles,
                               double* gt, int* words, int* notpd, int* stalled, int looks)
{
    const int T = (d + NB - 1) / NB, wgs = flow_grid(cus, 2 * (int64_t)T * T);
    const FlowInverseP p = inverse_params(H, d, damp, damp_abs, Hinv, tiles, gt, words, notpd, stalled, looks, wgs);
    hipLaunchKernelGGL(flow_inverse_kernel, dim3(wgs), dim3(NT), 0, s, p);
    return hipGetLastError();
}

// What the queues of an elimination have to do, in units of 2.3 us, a rank-64 product of a tile near the chain: tiles of U; parts of
// columns (3, 5 and 8 units for 1, 2 and 4 rows per wavefront; of a layer narrower than a block their steps are fewer); sums of 64 rows.  Where there are more groups of
// rows than blocks, the launch consists of parts and sums, and a sum is its products (1.5 units: their tiles come from farther
// away) and, whatever their number, a ticket, the gather of its weights and its publication (5 us).  Otherwise the products
// alone: queue 1's workgroups are free for the rest in the later half.  The best share of queue 3 in what queues 2 and 3 have,
// measured / by these: 65535 x 64 from 0.16 on / 0.16, 65535 x 512 0.30 / 0.34, 4000 x 1024 0.46 / 0.47, 8000 x 2048 0.69 / 0.62;
// 4096 x 4608 0.68 / 0.69 (6.80 ms; at 0.76 6.99), 2048 x 4608 0.70 to 0.76 / 0.69.  (With the products alone counted everywhere
// 8 workgroups had the sums of 65535 x 64 and 245 waited for them: 986 us for the layer, 666 with a launch per block, 580 so.)
// A part of 4 rows has become shorter since, 6.4 units; with 8, 7.2 and 6.4 the layer takes, 65535 x 512 2286, 2343, 2396 us, 20000 x 512 775,
// 782, 796, 4096 x 4608 5781, 5795, 5865, 8192 x 256 264, 264, 265, 2048 x 4608 4193, 4147, 4148, 30000 x 1500 3906, 3849, 3827.
static double work_u(double T) { return T * T * T / 6.0; }
static double work_columns(double T, double NG, int nr, int d)
{
    return T * NG * (8 / nr) * (nr == 1 ? 3.0 : nr == 2 ? 5.0 : 8.0) * (0.3 + 0.7 * d / (64.0 * T));
}
static double work_groups(double T, double NG) { return NG * T * (NG > T ? 0.75 * T + 2.2 : 0.5 * T); }

FlowElimPlan flow_eliminate_plan(int cus, int d, int R)
{
    // Where the chain of the diagonal blocks bounds the launch: what keeps up with it (two rows of tiles on queue 1, which feeds
    // everything else; half as many again as there are parts in a block; the groups' sums a few blocks ahead), and no more, so
    // that other launches find compute units.  Otherwise all, in proportion to the work of the queues.
    FlowElimPlan p;
    const int64_t T = (d + NB - 1) / NB, NG = (R + NB - 1) / NB;
    p.nr = column_rows(cus, R, T);
    const int64_t parts = NG * (8 / p.nr);
    // (a third more for queue 1 than its work: its workgroups go over to the other queues when it is empty, and those wait for its
    // rows until then.  The layer with 1, 1.15, 1.3, 1.5 and 1.7 times the work: 2048 x 4608 4355, 4255, 4217, 4204, 4337 us, 1024 x 3072 1661,
    // 1635, 1618, 1606, 1626, 512 x 4096 2500, 2498, 2500, 2504, 2583; 1000 x 2048, 2048 x 2048, 300 x 4608 and tall ones the same to 0.5 %)
    const double w1 = 1.3 * work_u((double)T), w2 = work_columns((double)T, (double)NG, p.nr, d), w3 = work_groups((double)T, (double)NG);
    const int64_t k1 = 2 * T, k2 = parts + (parts + 1) / 2, k3 = NG + NG * T / 6;
    const int avail = flow_grid(cus, T * (T + 9 * NG)) - 1;
    if (k1 + k2 + k3 <= avail) {
        p.n1 = (int)k1; p.n2 = (int)k2; p.n3 = (int)k3;
    } else {
        p.n1 = std::max<int>((int)(avail * w1 / (w1 + w2 + w3)), (int)std::min<int64_t>(k1, avail / 3));
        p.n1 = std::max(1, std::min(p.n1, avail - 2));
        p.n2 = std::max(1, std::min(avail - p.n1 - 1, (int)((avail - p.n1) * w2 / (w2 + w3) + 0.5)));
        p.n3 = avail - p.n1 - p.n2;
    }
    return p;
}

hipError_t launch_flow_eliminate(hipStream_t s, int cus, const FlowElimArgs& a)
{
    FlowElimP p = eliminate_params(a);
    const FlowElimPlan plan = flow_eliminate_plan(cus, a.d, a.R);
    const int nr = plan.nr;
    p.f.n1 = plan.n1; p.f.n2 = plan.n2; p.f.n3 = plan.n3;
    const int wgs = 1 + p.f.n1 + p.f.n2 + p.f.n3;
    switch (nr) {
    case 1: hipLaunchKernelGGL(flow_eliminate_kernel<1>, dim3(wgs), dim3(NT), 0, s, p); break;
    case 2: hipLaunchKernelGGL(flow_eliminate_kernel<2>, dim3(wgs), dim3(NT), 0, s, p); break;
    default: hipLaunchKernelGGL(flow_eliminate_kernel<4>, dim3(wgs), dim3(NT), 0, s, p); break;
    }
    return hipGetLastError();
}

// ---- several small layers (fobq_quantize_layers_batched) ----------------------------------------------------------
// A layer of at most 4 blocks is bound by its chain (12 to 14 us a block; an inverse of 1, 2, 3 and 4 blocks 37, 52, 64 and 76 us as a call); the
// layers' chains run side by side, and the launch ends when the device has worked off the parts of the longest ones.  20
// layers of 64 .. 1024 rows and 64 .. 256 columns: inverse 66 us (one workgroup per layer, a panel at a time: 311),
// elimination with columns 150 us (191 + 311 before, in launches of their own); the call 319 us, 1033 before.
static_assert(sizeof(FlowInverseP) <= FLOW_DESC_BYTES && sizeof(FlowElimP) <= FLOW_DESC_BYTES, "descriptor size");
constexpr int BATCH_INVERSE_WGS = 8;      // a layer of 4 blocks: the chain, and 25 tiles of R, X and Hinv

int flow_batch_most_wgs(int cus, int n) { return cus + n * (BATCH_INVERSE_WGS + 8); }

// How the workgroups of the batched elimination are dealt, and the rows per wavefront (the same for all layers).
void flow_batch_deal(int cus, int n, const int* d, const int* R, FlowElimPlan* out)
{
    // Rows per wavefront: the longest chains against twice the pure work over the device (see column_rows).
    double least = 0.0, total = 0.0;
    int nr = 1;
    for (int i = 0; i < 3; ++i) {
        double chains = 0.0, work = 0.0;
        for (int l = 0; l < n; ++l) {
            const double T = (d[l] + NB - 1) / NB, NG = (R[l] + NB - 1) / NB;
            chains = std::max(chains, T * std::max(BLOCK_US, PART_US[i] + 2.5));
            work += T * NG * (8 >> i) * PART_US[i] * 2.0 / (cus - 1);
        }
        const double time = std::max(chains, work);
        if (i == 0 || time < least) { least = time; nr = 1 << i; }
    }
    int fixed = 0;
    for (int l = 0; l < n; ++l) {
        const int T = (d[l] + NB - 1) / NB, NG = (R[l] + NB - 1) / NB;
        total += (double)T * NG;
        fixed += 1 + std::min(T, 4) + std::min(NG, 4);
    }
    // the device's workgroups, less those that every layer needs, in proportion to the layers' blocks of rows and columns; of a
    // layer's, what the sums of its rows want beyond the four (by work: one layer of 16000 x 256 1494 us with four, 1159 with
    // a launch per stage, 490 so)
    const int budget = std::max(cus - fixed, n);
    for (int l = 0; l < n; ++l) {
        const int T = (d[l] + NB - 1) / NB, NG = (R[l] + NB - 1) / NB, parts = NG * (8 / nr);
        const int base = std::min(NG, 4), share = (int)(budget * (double)T * NG / total);
        const double w2 = work_columns(T, NG, nr, d[l]), w3 = work_groups(T, NG);
        const int more = std::max(0, std::min(std::min((int)((base + share) * w3 / (w2 + w3)), NG) - base, share - 1));
        out[l].nr = nr;
        out[l].n1 = std::min(T, 4);
        out[l].n2 = std::max(1, std::min(parts, share - more));
        out[l].n3 = base + more;
    }
}

void flow_batch_plan(int cus, int n, const FlowElimArgs* a, const double* const* H, double damp, double damp_abs, int* const* words, void* inv_desc,
                     void* elim_desc, uint16_t* inv_of, uint16_t* elim_of, int* const* notpd_h, FlowBatchPlan* plan)
{
    FlowElimPlan deal[BATCH_MAX_LAYERS];
    int ds[BATCH_MAX_LAYERS], Rs[BATCH_MAX_LAYERS];
    for (int l = 0; l < n; ++l) { ds[l] = a[l].d; Rs[l] = a[l].R; }
    flow_batch_deal(cus, n, ds, Rs, deal);
    plan->nr = deal[0].nr;
    plan->inv_wgs = plan->elim_wgs = 0;
    for (int l = 0; l < n; ++l) {
        const int T = (a[l].d + NB - 1) / NB;
        const int wi = std::min(1 + 2 * T * T, BATCH_INVERSE_WGS);
        const FlowInverseP ip = inverse_params(H[l], a[l].d, damp, damp_abs, const_cast<double*>(a[l].Hinv), a[l].tiles, a[l].gt, words[l], notpd_h[l],
                                               a[l].stalled, a[l].looks, wi);
        memcpy(static_cast<unsigned char*>(inv_desc) + (size_t)l * sizeof(FlowInverseP), &ip, sizeof ip);
        for (int w = 0; w < wi; ++w) inv_of[plan->inv_wgs++] = (uint16_t)l;
        FlowElimP ep = eliminate_params(a[l]);
        ep.f.n1 = deal[l].n1; ep.f.n2 = deal[l].n2; ep.f.n3 = deal[l].n3;
        memcpy(static_cast<unsigned char*>(elim_desc) + (size_t)l * sizeof(FlowElimP), &ep, sizeof ep);
        for (int w = 0; w < 1 + ep.f.n1 + ep.f.n2 + ep.f.n3; ++w) elim_of[plan->elim_wgs++] = (uint16_t)l;
    }
}

hipError_t launch_flow_batch_inverse(hipStream_t s, const void* desc, const uint16_t* layer_of, int* arrivals, int wgs)
{
    hipLaunchKernelGGL(flow_inverse_batch_kernel, dim3(wgs), dim3(NT), 0, s, static_cast<const FlowInverseP*>(desc), layer_of, arrivals);
    return hipGetLastError();
}

hipError_t launch_flow_batch_eliminate(hipStream_t s, const void* desc, const uint16_t* layer_of, int* arrivals, int wgs, int nr)
{
    const FlowElimP* d = static_cast<const FlowElimP*>(desc);
    switch (nr) {
    case 1: hipLaunchKernelGGL(flow_eliminate_batch_kernel<1>, dim3(wgs), dim3(NT), 0, s, d, layer_of, arrivals); break;
    case 2: hipLaunchKernelGGL(flow_eliminate_batch_kernel<2>, dim3(wgs), dim3(NT), 0, s, d, layer_of, arrivals); break;
    default: hipLaunchKernelGGL(flow_eliminate_batch_kernel<4>, dim3(wgs), dim3(NT), 0, s, d, layer_of, arrivals); break;
    }
    return hipGetLastError();
}

}  // namespace fobq
