// Internal declarations shared by the translation units of libfobq (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string>
#include <vector>

#include "fobq.h"

namespace fobq {

// code = clamp(rint(w / scale) + zero, 0, maxq), rint = round half to even, all fp64 (Section 3: the fixed grid)
__device__ __forceinline__ double grid_code(double w, double scale, double zero, double maxq)
{
    double c = rint(w / scale) + zero;
    c = c < 0.0 ? 0.0 : c;
    c = c > maxq ? maxq : c;
    return c;
}

// The sum of n values a stride apart, in their order, four loads in flight (one thread, the entry's values in the slabs: a load at a
// time is its latency n times over: 512 rows with 61 slabs 250 -> 241 us for the whole call, 147 rows from maps 248 -> 243).
__device__ __forceinline__ double slab_sum(const double* __restrict__ p, int n, int64_t stride)
{
    double s = 0.0;
    int k = 0;
    for (; k + 4 <= n; k += 4, p += 4 * stride) {
        const double a = p[0], b = p[stride], c = p[2 * stride], e = p[3 * stride];
        s += a; s += b; s += c; s += e;
    }
    for (; k < n; ++k, p += stride) s += *p;
    return s;
}

// Entry (a, b) of a symmetric matrix of d columns and its mirror image, into H and, if there is one, H2: a workgroup of 256 has a tile of 16 x 16,
// row threadIdx.x / 16, whose lower triangle alone counts on the diagonal.  TURN: the tile changes places in LDS, so that the mirror image is
// written 16 entries a row as well (every thread of the workgroup comes here).  Without, a store instruction takes 16 pieces of 4 entries there,
// twice since H2 is written beside H: 4607 x 700 421 -> 424 us against a copy behind the launch, so 412; 4096 x 600 290, 279, 249; the
// barrier costs 1 us where the launch takes 4, up to 256 columns.
template <bool TURN>
__device__ __forceinline__ void store_symmetric(double s, int d, double* __restrict__ H, double* __restrict__ H2)
{
    const int x = threadIdx.x & 15, y = threadIdx.x >> 4;
    auto put = [&](int row, int col, double v) {
        H[(int64_t)row * d + col] = v;
        if (H2) H2[(int64_t)row * d + col] = v;
    };
    const int a = 16 * blockIdx.y + y, b = 16 * blockIdx.x + x;
    if (a < d && b <= a) put(a, b, s);
    if constexpr (TURN) {
        __shared__ double t[16 * 17];
        t[y * 17 + x] = s;
        __syncthreads();
        const int a2 = 16 * blockIdx.y + x, b2 = 16 * blockIdx.x + y;
        if (a2 < d && b2 <= a2) put(b2, a2, t[x * 17 + y]);
    } else if (a < d && b <= a) {
        put(b, a, s);
    }
}

// Looks that a wavefront inside a factorization launch waits while nobody in that launch draws a tile before the launch is given
// up.  A look takes 0.16 to 0.19 us (measured, one workgroup or 256 of them waiting): 43 to 51 seconds.
constexpr int FLOW_LOOKS = 1 << 28;

// ---------------------------------------------------------------------------
// Device buffer owned by the context; grows, never shrinks.
struct DevBuf {
    void*  p = nullptr;
    size_t cap = 0;
    hipError_t ensure(size_t bytes) {
        if (bytes <= cap) return hipSuccess;
        if (p) { (void)hipFree(p); p = nullptr; cap = 0; }
        size_t want = (bytes + 255) & ~size_t(255);
        hipError_t e = hipMalloc(&p, want);
        if (e == hipSuccess) cap = want; else p = nullptr;
        return e;
    }
    void release() { if (p) (void)hipFree(p); p = nullptr; cap = 0; }
    template <class T> T* as() const { return reinterpret_cast<T*>(p); }
};

// ---------------------------------------------------------------------------
// fp64 MFMA GEMM:  C = beta*C + alpha * op(A) * B, row-major.
//   op(A) is M x K:  TA=false -> A[m*lda + k],  TA=true -> A[k*lda + m];  B is K x N
// Tiles of 64 x 64 per workgroup; `upper`: only those on or above the diagonal.
struct GemmP {
    int M = 0, N = 0, K = 0;
    const double* A = nullptr; int64_t lda = 0;
    const double* B = nullptr; int64_t ldb = 0;
    double* C = nullptr;       int64_t ldc = 0;
    double* C2 = nullptr;              // optional second output: rowscale[m] * result
    const double* rowscale = nullptr;
    double alpha = 1.0, beta = 0.0;
    bool upper = false;
};
hipError_t gemm64(hipStream_t s, const GemmP& p, bool TA);

// `done` (in the launchers below that take one; may be null): an event that is recorded when the launch
// completes.  It rides on the launch as its stop event (hipExtLaunchKernelGGL): a separate hipEventRecord
// between two dependent launches is a bubble of about 4 us on the stream.

// ---------------------------------------------------------------------------
// Stage timing (hipEvents on the context's stream), off by default.
struct StageTimer {
    std::vector<std::pair<hipEvent_t, hipEvent_t>> pending[FOBQ_STAGE_COUNT];
    std::vector<hipEvent_t> pool;
    double  ms[FOBQ_STAGE_COUNT] = {0};
    int64_t launches[FOBQ_STAGE_COUNT] = {0};
};

}  // namespace fobq

constexpr int FLAG_WORDS = 16, FLAG_WORD_NONFINITE = 9;

struct fobq_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    std::string err;

    // Hessian accumulation state
    int64_t h_d = 0;        // d_col of the running accumulation (0 = none)
    int64_t h_n = 0;        // calibration columns seen so far
    int     h_splits = 0;   // split-K partial slabs in Hpart
    int     h_zeroed = 0;   // slabs of Hpart cleared (and possibly written) since hessian_begin
    bool    h_final = false;
    int     h_conv_c = 0;   // > 0: accumulation in convolution mode with this many channels ...
    int     h_conv_k = 0;   // ... and this kernel size; -1 in h_conv_c: plain mode
    int     h_mode = 0;     // fobq_hessian_mode
    bool    h_i8_used = false;  // the integer-slice kernels ran in this accumulation
    bool    h_offsets = false;  // convolution mode by tap offsets (hessian_offsets.hip) in this accumulation
    fobq::DevBuf hcorr;     // d x d fp64: the corrections of that mode, tap-major
    fobq::DevBuf strips;    // jobs x c x c fp64: the strips of one call
    fobq::DevBuf i8planes;  // digits of one accumulate call (see hessian_i8.hip)
    fobq::DevBuf i8sh;      // per-row shifts of that call
    fobq::DevBuf i8amax;    // per-channel maxima (convolution input)
    fobq::DevBuf batch_pool;    // scratch of all layers of a batched call
    fobq::DevBuf batch_desc;    // descriptors and workgroup tables of a batched call
    void* h_batch = nullptr;    // pinned host staging for the descriptors and the status read-back

    fobq::DevBuf Hpart;     // h_splits x d x d fp64 partial sums of X X^T (lower tiles)
    fobq::DevBuf maps_pad;  // zero-padded copy of the feature maps of one accumulate_conv call (+ 1 zero image)
    fobq::DevBuf H;         // d x d fp64, (2/N) X X^T, full symmetric

    // factorization / elimination workspace (all d x d fp64 unless noted)
    fobq::DevBuf tiles, gt; // published tiles of a factorization and its transposed block inverses (see flow.hip)
    fobq::DevBuf words;     // words of the two launches, then d_row fp64 per-row loss terms (lossrow); cleared per layer
    double* lossrow = nullptr;
    int* words2 = nullptr;  // the elimination's words inside that buffer
    int64_t words_len = 0;  // 4-byte words of that buffer in use
    fobq::DevBuf tilesN;    // a second set of published tiles (Un of the elimination)
    fobq::DevBuf vec;       // 128 fp64 per 64 columns: reciprocal pivots, half reciprocal pivots
    fobq::DevBuf Hinv;
    fobq::DevBuf A, U, Un;  // general elimination (block != 64, or not all columns)
    fobq::DevBuf Dblk;      // general elimination: one block's G (64 x 64) and 64 reciprocal pivots
    fobq::DevBuf obq;       // running inverses of the per-row baseline (fobq_obq_rows), rows x d x d fp64
    fobq::DevBuf flags;     // FLAG_WORDS int32: status flags written by kernels (cleared per call), then words
                            // that live longer (FLAG_WORD_NONFINITE: an accumulation)
    int cus = 256;          // compute units of the device (fobq_create)
    int* h_flags = nullptr; // pinned host memory that the status flags are read back into (made by fobq_create)
    bool flags_sent = false;    // the enqueued layer's last launch writes them there itself
    unsigned char* static_scratch = nullptr;   // this GPU's copy of the library's static scratch array
    int flow_looks = fobq::FLOW_LOOKS;   // (test hook: fobq_debug_wait_looks)
    int fail_countdown = 0; // test hook: > 0 = the n-th status check from now reports an injected failure
    // quantization workspace
    fobq::DevBuf Wp;        // d_row x d fp64, columns in processing order (one-launch form: in tiles)
    fobq::DevBuf DT;        // d x Rp fp64: (w - q) per processed column (one-launch form: in tiles)
    fobq::DevBuf corr;      // 2 x Rp x 64 fp64: compensation handed from one column block to the next
    fobq::DevBuf codesT;    // d x Rp u8
    fobq::DevBuf scale, zero;   // d_row x G fp64
    fobq::DevBuf S, Spart;  // d fp64, chunks x d fp64
    fobq::DevBuf perm, invperm; // d int32

    // second stream: the column loop of block k only needs the pivot rows of blocks <= k, so it
    // runs behind the shared-Hinv elimination on its own stream, ordered by one event per block
    hipStream_t side = nullptr;
    int side_missed = 0;    // calls that would have used it and kept to the context's stream
    std::vector<hipEvent_t> sync_ev;

    bool pending = false;   // a layer was enqueued without the final status read (fobq_finish outstanding)
    unsigned profiling = 0;     // bit s: stage s is timed
    fobq::StageTimer timer;
};

namespace fobq {

// One layer of fobq_quantize_layers_batched as the kernels see it (an array of these lives in device memory).
// All pointers are device memory; the scratch pointers are carved out of one pool of the context.
struct BatchLayer {
    const float* W; const double* H;          // inputs
    int R, d, G, gs, Rp, chunks;              // G grids per row of gs columns; Rp = R rounded up to 64; chunks = sens_chunks(R)
    double maxq;
    int order, kind, ascending;               // fobq_order; sort key (0 sensi, 1 err, 2 w); direction
    double *Hinv;                             // d x d
    double *tiles, *tilesN, *gt, *vec, *wt, *dt, *corr;   // scratch of the two factorization launches (see FlowElimArgs)
    int *words; int nwords, nwords1;          // their words: nwords in all, the inverse's nwords1 first,
                                              // last the launches' two counts of workgroups (used: layer 0's)
    uint8_t* codesT;                          // d x Rp
    double *scale, *zero;                     // R x G
    double *S, *Spart, *lossrow;              // d; chunks x d; R
    int *perm, *invperm, *flags;              // d; d; 4 status words (as FLAG_* of a single layer)
    uint8_t* codes; float *scales, *zeros, *Q; int* perm_out; double* loss;   // outputs (may be null)
};
constexpr int BATCH_MAX_D = 256;      // columns of a layer in a batched call (4 panels of 64)
constexpr int BATCH_MAX_LAYERS = 256;

int set_err(fobq_ctx* c, int code, const char* fmt, ...);
int hip_err(fobq_ctx* c, hipError_t e, const char* what);

// Timing of a stage that is exactly one launch: the two events ride on the launch as its start and stop
// events (no bubble on the stream; StageScope's records cost about 4 us each).  Both null when the stage is
// not being timed.
struct LaunchEvents { hipEvent_t start = nullptr, stop = nullptr; };
LaunchEvents stage_launch_events(fobq_ctx* c, int stage);

struct StageScope {
    fobq_ctx* c; int stage; hipStream_t st; hipEvent_t e0 = nullptr, e1 = nullptr;
    StageScope(fobq_ctx* c_, int stage_, hipStream_t on = nullptr);   // on == nullptr: the context's stream
    ~StageScope();
};

// hessian.hip; fresh: 0, or on the first launch of an accumulation the slabs that it then has (xxt_slabs_touched), which need
// not hold anything before
hipError_t launch_xxt(hipStream_t s, const float* X, int64_t ld, int d, int64_t n, double* Hpart, int splits, int fresh,
                      LaunchEvents ev = LaunchEvents());
int xxt_pick_splits(int d);
int xxt_tile(int d, int64_t n);       // tile edge of a launch over n calibration columns
int xxt_slabs_touched(int d, int64_t n, int splits, bool conv);
hipError_t launch_clear_slabs(hipStream_t s, double* Hpart, int d, int first, int count);
// the padding launch: `parts` runs of `run` pixels (the last one the rest) of each of `rows` rows, wgs workgroups of 256 threads; whether it moves 16 bytes per lane and takes
// the channel maxima along
struct PadPlan { int64_t rows; int parts, run, wgs, active; bool vec, maxima; };
PadPlan pad_maps_plan(int64_t n_img, int h, int w, int c, int pad, bool aligned, bool maxima);
hipError_t launch_pad_maps(hipStream_t s, const float* maps, int n_img, int h, int w, int c, int pad, float* out, unsigned* amax, bool* took,
                           hipEvent_t done = nullptr);
hipError_t launch_xxt_conv(hipStream_t s, const float* padded, int n_img, int hp, int wp, int c, int k, int stride,
                           int ho, int wo, int64_t npix, double* Hpart, int splits, int fresh,
                           LaunchEvents ev = LaunchEvents());
// (H2: null, or a second place for H)
hipError_t launch_hessian_finalize(hipStream_t s, double* Hpart, int splits, int d, double factor, double* H, double* H2,
                                   int conv_c, int conv_kk, const int* poison);   // *poison != 0: H = NaN

// hessian_i8.hip: X X^T by exact integer slices on the int8 matrix cores
int i8_dpad(int d);
size_t i8_planes_bytes(int d, int64_t n);
// rect.cb > 0: instead of the lower triangle, tiles of two groups of rect.cb tile rows (the second group starts at tile row
// rect.gap), which hold the rows of the taps (0, 0) and (0, k - 1) of a convolution of c64 * 64 channels: those tiles that
// hold a block of a pair of taps that the assembly by tap offsets reads (i8_rect_needs).  rect.half (with cb = gap = 1): the two
// groups are the first 64 rows of tile rows 0 and 1 only, and one tile row made of those 128 rows is formed instead of two, all
// its tile columns.
struct I8Rect { int cb = 0, gap = 0, half = 0, c64 = 0, k = 0; };
// Whether tile (I, J) is formed.  In blocks of 64 rows and columns: from tap (0, 0) the offsets that point right or down, to any
// tap, of the zero offset the triangle on and below the diagonal; from tap (0, k - 1) those that point left and down, to the taps
// of the other map rows left of its column.  256 channels, 3 x 3: 51 tiles instead of the 72 of the rows, the call 704 -> 630 us.
__host__ __device__ inline bool i8_rect_needs(const I8Rect& r, int I, int J)
{
    for (int a = 2 * I; a < 2 * I + 2; ++a)
        for (int b = 2 * J; b < 2 * J + 2; ++b) {
            const int ta = a / r.c64, tb = b / r.c64;
            if (tb >= r.k * r.k) continue;
            if (ta == 0 ? tb > 0 || b <= a : ta == r.k - 1 && tb >= r.k && tb % r.k < r.k - 1) return true;
        }
    return false;
}
// full > 0: the workgroups go through the tiles in step (see xxt_i8_kernel): `full` rounds of whole tiles, then the
// `rem` tiles left over, each cut into `pieces` parts of piece_len k-steps
struct I8Lockstep { int full = 0, rem = 0, pieces = 0; int64_t piece_len = 0; };
int xxt_i8_slabs_touched(int d, int64_t n, int splits, I8Rect rect = I8Rect());
// slabs of partial sums that a launch over n columns would like to have (0: no wish beyond xxt_pick_splits)
int xxt_i8_wanted_splits(int d, int64_t n, I8Rect rect = I8Rect());
int64_t i8_block_columns(int d);      // most columns one launch of the matrix kernel takes (bounds the digit scratch)
hipError_t launch_i8_row_shifts(hipStream_t s, const float* X, int64_t ld, int d, int64_t n, int* sh, int* nonfinite);
hipError_t launch_i8_slice(hipStream_t s, const float* X, int64_t ld, int d, int64_t n, const int* sh, signed char* planes);
hipError_t launch_i8_chan_shifts(hipStream_t s, const float* padded, int64_t pixels, int c, int d, unsigned* amax, bool have_amax,
                                 int* sh, int* nonfinite);
hipError_t launch_i8_slice_conv(hipStream_t s, const float* padded, int n_img, int hp, int wp, int c, int k, int stride,
                                int ho, int wo, int64_t npix, int64_t pix0, int64_t n, const int* sh, signed char* planes);
hipError_t launch_xxt_i8(hipStream_t s, const signed char* planes, const int* sh, int d, int64_t n, double* Hpart,
                         int splits, int fresh, LaunchEvents ev = LaunchEvents(), I8Rect rect = I8Rect());   // fresh: as for launch_xxt
// hessian_offsets.hip: Hessian of a stride-1 convolution by tap offsets (two block rows from the digit-product kernel,
// the other blocks by corrections over single rows and columns of the padded maps)
constexpr int OFFSET_MAX_TAPS = 9, OFFSET_MAX_JOBS = 128, OFFSET_MAX_PAIRS = 81, OFFSET_MAX_TERMS = 384;
// one strip: kind 0 = row `coord` of the padded map, columns start .. start + len - 1; kind 1 = column `coord`, rows
// start .. start + len - 1; (dy, dx) = the offset of the second factor
struct OffsetJob { int coord, start, len; signed char kind, dy, dx, unused; };
// passed to the kernels by value (about 3 KiB)
struct OffsetTables {
    int njobs, npairs, nterms;
    OffsetJob jobs[OFFSET_MAX_JOBS];
    unsigned char pair_ta[OFFSET_MAX_PAIRS], pair_tb[OFFSET_MAX_PAIRS];   // tap indices ky * k + kx of a pair with corrections
    short pair_begin[OFFSET_MAX_PAIRS + 1];                               // its terms: [pair_begin[p], pair_begin[p + 1])
    unsigned char term_job[OFFSET_MAX_TERMS];
    signed char term_sign[OFFSET_MAX_TERMS];
};
bool offset_tables_build(int k, int pad, int h, int w, OffsetTables* tab);
size_t offset_strips_bytes(int njobs, int c);
hipError_t launch_clear_slab_rows(hipStream_t s, double* Hpart, int d, int first, int count, int row0, int n0, int row1, int n1);
// (both only where the tables have jobs)
hipError_t launch_offset_strips(hipStream_t s, const float* padded, int n_img, int hp, int wp, int c, const OffsetTables& tab, double* strips);
hipError_t launch_offset_apply(hipStream_t s, int c, int d, const OffsetTables& tab, const double* strips, double* corr, hipEvent_t done);
hipError_t launch_hessian_finalize_offsets(hipStream_t s, const double* Hpart, int splits, int d, double factor, double* H, double* H2, int c,
                                           int k, const double* corr, const int* poison);

// flow.hip: damped H -> upper tiles of Hinv = (H + lambda I)^-1, lambda = damp * mean(diag H) + damp_abs, in one launch.  tiles, gt:
// scratch; words: flow_inverse_words(d) zeroed words; *notpd / *stalled are set to 1 when a pivot is not positive / the launch gave up
// after `looks` looks of a waiting wavefront during which nobody drew a tile (FLOW_LOOKS)
int64_t flow_inverse_words(int d);
size_t flow_tiles_bytes(int d);
size_t flow_gt_bytes(int d);
// The shared-Hinv elimination and the column loop of a whole layer in one launch.  words: flow_eliminate_words(cus, d, R) zeroed words;
// tiles, tilesN: flow_tiles_bytes(d); gt: flow_gt_bytes(d); vec: 128 doubles per 64 columns; wt, dt: flow_rows_bytes(d, R);
// corr: 2 x Rp x 64; lossrow: zeroed; Wout may be null.
struct FlowElimArgs {
    int d, R, G, gs, bits, Rp;
    const double* Hinv; const int* perm; const float* W; const double *scale, *zero;
    double *tiles, *tilesN, *gt, *vec, *wt, *dt, *corr, *lossrow, *Wout;
    uint8_t* codesT;
    int *words, *notpd, *stalled;
    int looks;
};
int64_t flow_eliminate_words(int cus, int d, int R);
int64_t flow_eliminate_words_most(int d, int R);     // however many rows a wavefront takes
size_t flow_rows_bytes(int d, int R);
// rows per wavefront of a part of columns, and the workgroups that serve each queue first
struct FlowElimPlan { int nr, n1, n2, n3; };
FlowElimPlan flow_eliminate_plan(int cus, int d, int R);
void flow_batch_deal(int cus, int n, const int* d, const int* R, FlowElimPlan* out);
hipError_t launch_flow_eliminate(hipStream_t s, int cus, const FlowElimArgs& a);
hipError_t launch_flow_inverse(hipStream_t s, int cus, const double* H, int d, double damp, double damp_abs, double* Hinv, double* tiles,
                               double* gt, int* words, int* notpd, int* stalled, int looks);

// factor.hip
// `rows_ready` (may be null): rows_ready[k] is recorded on the context's stream once the pivot rows of
// block k (rows k*block .. of U and Un) are complete (hipEventRecord: about 4 us on the stream, in a path of three launches a
// block).
hipError_t eliminate_blocked(fobq_ctx* c, double* A, int d, int steps, int block, double* U, double* Un, int* flag,
                             const std::vector<hipEvent_t>* rows_ready);

// several small layers in one launch of each kind: descriptors (FLOW_DESC_BYTES each at most, packed as the kernels read them) and
// the layer of every workgroup, for both launches
constexpr size_t FLOW_DESC_BYTES = 320;
struct FlowBatchPlan { int inv_wgs, elim_wgs, nr; };
int flow_batch_most_wgs(int cus, int n);
void flow_batch_plan(int cus, int n, const FlowElimArgs* a, const double* const* H, double damp, double damp_abs, int* const* words, void* inv_desc,
                     void* elim_desc, uint16_t* inv_of, uint16_t* elim_of, int* const* notpd_h, FlowBatchPlan* plan);
hipError_t launch_flow_batch_inverse(hipStream_t s, const void* desc, const uint16_t* layer_of, int* arrivals, int wgs);
hipError_t launch_flow_batch_eliminate(hipStream_t s, const void* desc, const uint16_t* layer_of, int* arrivals, int wgs, int nr);

// the rest of a batched call: quant.hip; grids have one dimension over the layers
hipError_t launch_batch_order(hipStream_t s, const BatchLayer* layers, int n);
hipError_t launch_batch_grid(hipStream_t s, const BatchLayer* layers, int n, int max_pairs, hipEvent_t done);
hipError_t launch_batch_sens_partial(hipStream_t s, const BatchLayer* layers, int n, int max_chunks, hipEvent_t done);
hipError_t launch_batch_emit(hipStream_t s, const BatchLayer* layers, int n, int max_tiles);   // max_tiles: of 16 rows x 64 columns

// per-row baseline (obq.hip)
constexpr int OBQ_MAX_D = 4096;        // columns: a row's weights, pivot row and flags live in LDS
size_t obq_scratch_per_row(int d);
hipError_t launch_obq_rows(hipStream_t s, const float* W, int d, int bits, int group, const double* Hinv0, const double* scale,
                           const double* zero, int row_begin, int rows, double* Hscratch, uint8_t* codes, float* Q, int* order,
                           double* lossrow, int* flag);

// quant.hip
hipError_t launch_grid(hipStream_t s, const float* W, int R, int d, int bits, int group,
                       double* scale, double* zero, float* scales_out, float* zeros_out);
hipError_t launch_sens_partial(hipStream_t s, const float* W, int R, int d, int bits, int group,
                               const double* scale, const double* zero, double* Spart, int chunks, int kind, hipEvent_t done = nullptr);
hipError_t launch_sens_reduce(hipStream_t s, const double* Spart, int chunks, int d, const double* Hinv, double* S,
                              int kind);
int sens_chunks(int R);
hipError_t launch_rank_sort(hipStream_t s, const double* S, int d, int* perm, int* invperm, int ascending);
hipError_t launch_iota(hipStream_t s, int d, int* perm, int* invperm);
hipError_t launch_check_perm(hipStream_t s, const int* perm_in, int d, int* perm, int* invperm, int* flag);
hipError_t launch_gather(hipStream_t s, const float* W, int R, int d, const int* perm,
                         const double* Hinv_upper, double* Wp, double* A, hipEvent_t done = nullptr);
hipError_t launch_col_block(hipStream_t s, double* Wp, int R, int d, int o, int nb,
                            const double* Un, const double* U, const double* scale, const double* zero,
                            int G, int group, const int* perm, int bits,
                            uint8_t* codesT, double* DT, int Rp, double* lossrow,
                            const double* corr_in, double* corr_out, int nb_next,
                            int uo, int unb, int c0, hipEvent_t done = nullptr);
hipError_t launch_invert_perm(hipStream_t s, const int* perm, int d, int* invperm);
hipError_t launch_dyn_select(hipStream_t s, double* Wp, int R, int d, int t, double* A, const double* scale,
                             const double* zero, int G, int group, int* perm, int bits, double* Spart, int chunks);
hipError_t launch_step(hipStream_t s, double* Wp, int R, int d, int t, double* A,
                       const double* scale, const double* zero, int G, int group, const int* perm, int bits,
                       uint8_t* codesT, int Rp, double* lossrow, int* flag);   // *flag = 1 when the pivot is not > 0
// what a layer's last launch does besides: the order to the caller (perm_out may be null), the status words to pinned host memory
struct EmitTail { const int* perm = nullptr; int* perm_out = nullptr; const int* flags = nullptr; int* host_flags = nullptr; int n_flags = 0; };
hipError_t launch_emit(hipStream_t s, const uint8_t* codesT, int Rp, int R, int d, int steps,
                       const int* invperm, const double* scale, const double* zero, int G, int group,
                       uint8_t* codes, float* Q, const double* lossrow, double* loss, EmitTail tail);   // loss may be null
hipError_t launch_loss(hipStream_t s, const double* lossrow, int R, double* loss);
hipError_t launch_hinv_work(hipStream_t s, const double* A, int d, int steps, double* out);
hipError_t launch_fill_i32(hipStream_t s, int* p, int64_t n, int v);
hipError_t launch_clear_words(hipStream_t s, void* p1, int64_t n1, void* p2, int64_t n2,
                              hipEvent_t done = nullptr);   // 4-byte words

}  // namespace fobq
