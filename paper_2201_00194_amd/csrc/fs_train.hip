// Training of family cost models: histogram boosting rounds on the device.
//
// After every tuning step the tuner retrains the family's model on the measured candidates
// (Algorithm 1 of the paper, train_cost_model; Section 4.3 moves this to the GPU).  The
// arithmetic is stated in familyseer_train.h.  What makes it reproducible bit for bit is that
// every sum over rows is an integer sum (gradients in fixed point, curvature = rows of the
// program), so the atomics below may land in any order; gains and leaf values are evaluated
// in double from those integers in one fixed order of operations.
//
// Per round and family (all families of a batch share every launch; nothing returns to the
// host between rounds):
//   grad         per program: s_p (row order), g_p, q_p; its rows' records (row, q_p, rows of p)
//                go back to the root; the root's (G, H) are added up on the way
//   hist, split  histograms and best cuts of the root
//   per level:   move (every workgroup decides its node for itself: best feature, split or leaf; the node's
//                records go to its children's segments, rows of leaves take the leaf's value), hist (LDS
//                histograms of the child with fewer rows, sixteen features per workgroup; the
//                other child is the parent minus that one, exactly; a feature's most frequent bin is
//                never counted, it is the node's total minus the rest) or, for few rows, both in one launch
//                (grow: from the parent's records, of the child with the smaller curvature, as the children's
//                rows are not counted yet); split (adds up the parts of nodes whose rows were dealt to several workgroups,
//                subtracts, searches the cuts of both children)
//   last level:  finish (decides its nodes; rows take the leaves' values)
//   (one more workgroup of the next round's first hist: heap -> flat model arrays, heap cleared)
#include <math.h>
#include <stdlib.h>
#include <string.h>
#include <algorithm>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

#include "familyseer_train.h"
#include "fs_internal.h"
#include "fs_lds.h"
#include "fs_runs.h"

namespace fs {

constexpr int kHeapNodes = (1 << (FS_TRAIN_MAX_DEPTH + 1)) - 1;   // 2047
constexpr int kBins = FS_TRAIN_MAX_CUTS + 1;                      // 256
constexpr int kHistFeats = 16;          // features per workgroup: 16 bytes of bins per row
constexpr int kHistWords = kHistFeats * kBins;
constexpr int kChunkShiftMin = 10;      // at least 1024 rows to a histogram workgroup: zeroing and storing its LDS
                                        // costs as much as 256 rows
constexpr int kChunkSmallRows = 12288;  // 2048 in batches of more rows than this: a round of depth 6 of 8500 / 12 700 /
                                        // 25 500 rows takes 93.9 / 99.8 / 115.0 us with 1024, 95.3 / 98.7 / 107.7 with 2048
constexpr int kMostGroups = 1024;       // items of so many rows as a batch has, times the feature groups of a workgroup
                                        // each: four fit a compute unit.  213 000 rows of five groups: 170 us a round with
                                        // 2048 rows, 175 with 4096; 308 000 of eleven: 286 with 2048, 280 with 4096, 297 with 8192

// heap node states (undecided or not in the tree: absent)
enum { kAbsent = 0, kInternal = 2, kLeaf = 3 };

// A (node, feature)'s best cut; cut 0 = none is admissible.
struct __align__(32) Best {
    double gain;
    int32_t cut;
    int32_t count_left;        // the left child is the counted one, see counts_left
    long long GL, HL;
};

// Sums over all rows of a round.
struct RootSums {
    // (lines of their own: every wavefront of the launch adds to each)
    __align__(128) long long G;
    __align__(128) long long H;
    __align__(128) unsigned long long abs_q;   // sum of |gradient| (fixed point)
};

struct TrainDesc {
    const uint8_t *bins;       // [row][row_bytes]: what a histogram workgroup gathers.  A row's features lie
                               // together so that the sixteen-byte pieces of all feature groups, taken by
                               // workgroups of one XCD, are a line or two of its L2 and not one line each
    const uint8_t *cols;       // [feature][r_pad]: the same by feature, for moving rows to a child
    const int32_t *prog_off;
    const float *target;
    const int32_t *cut_off;    // device copies of the cut lists
    const float *cuts;
    const int32_t *hot_bin;    // per feature: its most frequent bin, which no histogram counts
                               // (it is the node's total minus the other bins)
    float *row_pred;
    float *prog_pred;
    int4 *rec[2];              // {row, gradient in fixed point, curvature, output so far (bits)} of every row, grouped
                               // by the node of a level; levels alternate between the two
    int4 *seg;                 // per node of the heap: {rows gone left, rows gone right, first position, end}; no rows
                               // gone while the node is not split, no segment where there is no node.  The left child's
                               // records fill the segment from its front, the right child's from its back
    int32_t *h_slot;           // where in `hist` the node's histograms are
    unsigned long long *hist;  // [slot][feature][bin]: complete histograms, what the next level subtracts from
    unsigned long long *part;  // the same of parts of a node, see part_slot
    int64_t hist_plane, part_plane;   // words to the curvature sums (wide form)
    float *h_val;              // leaves of the deepest level
    long long *h_G, *h_H;
    double *h_own;             // the node's own term of the gain
    Best *best;                // [node of the level][feature]
    int4 *decision;            // per node of the heap: {state, feature, -, threshold or leaf value (bits)}
    int32_t *counters;         // [1] trees, [2] nodes, [3] rows of the longest program
    RootSums *root;            // two, rounds take them in turn: one is cleared while the other is in use
    int32_t *m_tree_off, *m_feat, *m_left, *m_right;
    float *m_thr, *m_val;
    int64_t r_pad;
    int32_t row_bytes;
    int32_t n_features, n_rows, n_programs;
    float bias;
};

// A trainer's descriptor as kernels read it: what a launch finds in constant memory are pointers to global memory, so that
// everything behind them is read by global and scalar loads.  (Through a plain pointer those were flat loads, which count as
// LDS reads too: waits for all of both kinds, one after the other, in launches that are chains of latencies.)
#if defined(__HIP_DEVICE_COMPILE__)
typedef __attribute__((address_space(4))) const TrainDesc Desc;
#else
typedef const TrainDesc Desc;
#endif

struct Params {
    double eta, lambda, min_gain, inv_scale;
    long long mcw;
    float grad_scale;
    int max_depth;
};

// ---- set-up kernels ----------------------------------------------------------------------

// Workgroups go to the eight XCDs in turn, and on an XCD to its compute units in turn.  A grid of
// (8 x feature groups, trainers, pieces / 8) takes the workgroups of a piece, one per feature group, to one XCD, one
// after the other, so that they share its L2.  The trainers' first eight pieces come first, then their next
// eight and so on: what a launch has too many of, being sized for the most pieces a trainer may have, ends up
// last.  (One trainer after the other left gaps between them, and compute units without work beside others
// with twice as much: two families of 34 000 rows of 250 features 190 us a round, so 180.)  A trainer's
// number moves its first piece to another XCD: families of five pieces would leave three XCDs idle.
__device__ __forceinline__ int xcd_piece(unsigned x, unsigned trainer, unsigned layer)
{
    return (int)(layer * 8 + ((x + 5 * trainer) & 7));
}

constexpr int64_t kMostPieces = 8 * 65535;     // of a trainer in one grid

// bin = number of cuts <= x; NaN takes the last bin.  A workgroup takes 256 rows of sixteen features,
// whose cut lists fit LDS together, so that a row's sixteen bins leave in one store.
__global__ void __launch_bounds__(256)
train_bin_kernel(const float *__restrict__ x, int layout, int n_features, int n_rows,
                 int64_t r_pad, const int32_t *__restrict__ cut_off,
                 const float *__restrict__ cuts, uint8_t *__restrict__ bins, int row_bytes,
                 uint8_t *__restrict__ cols)
{
    __shared__ float c[kHistFeats][kBins];
    const int groups = (n_features + kHistFeats - 1) / kHistFeats;      // a piece's to one XCD, as in xcd_piece
    const int layer = (int)(blockIdx.x >> 3) / groups, group = (int)(blockIdx.x >> 3) - layer * groups;
    const int64_t block = xcd_piece(blockIdx.x, 0, layer);
    if (block * blockDim.x >= n_rows)
        return;
    const int f0 = group * kHistFeats;
    const int nf = min(kHistFeats, n_features - f0);
    for (int i = threadIdx.x; i < kHistWords; i += blockDim.x) {
        const int f = min(f0 + i / kBins, n_features - 1), j = i % kBins;
        c[i / kBins][j] = j < cut_off[f + 1] - cut_off[f] ? cuts[cut_off[f] + j] : __builtin_inff();
    }
    __syncthreads();
    const int64_t r = block * (int64_t)blockDim.x + threadIdx.x;
    if (r >= n_rows)
        return;
    uint32_t w[kHistFeats / 4] = {};
#pragma unroll
    for (int k = 0; k < kHistFeats; ++k) {
        const int f = min(f0 + k, n_features - 1), m = cut_off[f + 1] - cut_off[f];   // (one load pattern for all)
        const float v = layout == FS_COLBLOCK64 ? x[(r >> 6) * n_features * 64 + (int64_t)f * 64 + (r & 63)]
                                                : x[r * n_features + f];
        int lo = 0;                              // cuts known to be <= v; entries past the list never are
#pragma unroll
        for (int step = kBins / 2; step > 0; step >>= 1)
            if (c[k][lo + step - 1] <= v)
                lo += step;
        lo = v != v ? m : min(lo, m);            // (+inf passes the padding too)
        if (k < nf) {
            w[k >> 2] |= (uint32_t)lo << (8 * (k & 3));
            cols[f * r_pad + r] = (uint8_t)lo;
        }
    }
    *(uint4 *)(bins + r * row_bytes + f0) = make_uint4(w[0], w[1], w[2], w[3]);
}

// Rows per (feature, bin): 8192 rows of a feature per workgroup, counted in LDS by each wavefront for itself.
constexpr int kCountRows = 8192;

__global__ void __launch_bounds__(256)
train_count_kernel(const uint8_t *__restrict__ cols, int n_rows, int64_t r_pad, uint32_t *__restrict__ count)
{
    __shared__ uint32_t cnt[4][kBins];
    const int t = threadIdx.x, f = blockIdx.y;
    for (int w = 0; w < 4; ++w)
        cnt[w][t] = 0u;
    __syncthreads();
    const int64_t first = blockIdx.x * (int64_t)kCountRows;
    const int n = (int)min((int64_t)kCountRows, n_rows - first);
    const uint32_t *words = (const uint32_t *)(cols + f * r_pad + first);   // r_pad and first are multiples of 256
#pragma unroll 4
    for (int i = 4 * t; i < n; i += 4 * 256) {
        const uint32_t v = words[i >> 2];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i + k < n)
                atomicAdd(&cnt[t >> 6][(v >> (8 * k)) & 255], 1u);
    }
    __syncthreads();
    const uint32_t all = cnt[0][t] + cnt[1][t] + cnt[2][t] + cnt[3][t];
    if (all != 0u)
        atomicAdd(&count[f * kBins + t], all);
}

// Largest of a workgroup's values, in thread 0.
__device__ int largest_of(int m)
{
    __shared__ int part[kBins / 64];
    for (int off = 32; off > 0; off >>= 1)
        m = max(m, __shfl_down(m, off));
    if ((threadIdx.x & 63) == 0)
        part[threadIdx.x >> 6] = m;
    __syncthreads();
    for (int w = 0; w < kBins / 64; ++w)
        m = max(m, part[w]);
    return m;
}

// What a new trainer starts with: the cut lists, if they are in pinned host memory (`staged`, n_words of them), no
// rows counted, no trees, every row's output the bias.  Each workgroup leaves the longest of its programs in `longest`.
__global__ void __launch_bounds__(kBins)
train_clear_kernel(const int32_t *__restrict__ staged, int n_words, int32_t *__restrict__ cut_off, uint32_t *count, int n_count,
                   int32_t *counters, int32_t *tree_off, float *row_pred, int64_t n_rows, float bias,
                   const int32_t *__restrict__ prog_off, int n_programs, int32_t *longest)
{
    const int64_t at = blockIdx.x * (int64_t)kBins + threadIdx.x, step = (int64_t)gridDim.x * kBins;
    if (staged)
        for (int64_t i = at; i < n_words; i += step)
            cut_off[i] = staged[i];
    for (int64_t i = at; i < n_count; i += step)
        count[i] = 0u;
    for (int64_t i = at; i < n_rows; i += step)
        row_pred[i] = bias;
    if (blockIdx.x == 0 && threadIdx.x < 3)
        counters[threadIdx.x] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 3)
        tree_off[0] = 0;
    int m = 0;
    for (int64_t p = at; p < n_programs; p += step)
        m = max(m, prog_off[p + 1] - prog_off[p]);
    m = largest_of(m);
    if (threadIdx.x == 0)
        longest[blockIdx.x] = m;
}

// The most frequent bin of every feature over the whole training set (lowest on ties).  A workgroup behind the last
// feature's finds the longest program (it sizes the curvature sums), also for the host (pinned memory, or null).
__global__ void __launch_bounds__(kBins)
train_hot_bin_kernel(const uint32_t *__restrict__ count, int n_features, int32_t *__restrict__ hot_bin,
                     const int32_t *__restrict__ longest, int n_longest, int32_t *__restrict__ max_len, int32_t *host_max_len)
{
    __shared__ unsigned int s_best[kBins];
    __shared__ int s_arg[kBins];
    const int f = blockIdx.x, t = threadIdx.x;
    if (f == n_features) {
        int m = 0;
        for (int i = t; i < n_longest; i += kBins)
            m = max(m, longest[i]);
        m = largest_of(m);
        if (t == 0) {
            *max_len = m;
            if (host_max_len)
                *host_max_len = m;
        }
        return;
    }
    s_best[t] = count[f * kBins + t];
    s_arg[t] = t;
    __syncthreads();
    for (int off = kBins / 2; off > 0; off >>= 1) {
        if (t < off) {
            const unsigned int a = s_best[t], b = s_best[t + off];
            if (b > a || (b == a && s_arg[t + off] < s_arg[t])) {
                s_best[t] = b;
                s_arg[t] = s_arg[t + off];
            }
        }
        __syncthreads();
    }
    if (t == 0)
        hot_bin[f] = s_arg[0];
}

// The model for the host, in pinned memory of `cap` words: trees, nodes, 1; the trees' offsets; the nodes' features,
// thresholds, children and values.  Without room for them the third word is 0.
__global__ void __launch_bounds__(256)
train_export_kernel(const TrainDesc d, int32_t *out, int64_t cap)
{
    const int64_t trees = d.counters[1], nodes = d.counters[2];
    const bool fits = 4 + trees + 1 + 5 * nodes <= cap;
    const int64_t at = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    if (at == 0) {
        out[0] = (int32_t)trees;
        out[1] = (int32_t)nodes;
        out[2] = fits ? 1 : 0;
    }
    if (!fits)
        return;
    out += 4;
    for (int64_t i = at; i <= trees; i += step)
        out[i] = d.m_tree_off[i];
    out += trees + 1;
    for (int64_t i = at; i < nodes; i += step) {
        out[i] = d.m_feat[i];
        out[nodes + i] = __float_as_int(d.m_thr[i]);
        out[2 * nodes + i] = d.m_left[i];
        out[3 * nodes + i] = d.m_right[i];
        out[4 * nodes + i] = __float_as_int(d.m_val[i]);
    }
}

// ---- per-round kernels -------------------------------------------------------------------

// The heap of the tree to grow and the sums of the round to come (one workgroup per trainer).  What belongs
// to a node below the root is written when its parent is split.
__device__ __forceinline__ void begin_tree(Desc &d, int turn)
{
    for (int i = threadIdx.x; i < kHeapNodes; i += blockDim.x) {
        d.decision[i] = make_int4(kAbsent, 0, 0, 0);
        d.seg[i] = make_int4(0, 0, 0, i == 0 ? d.n_rows : 0);
    }
    if (threadIdx.x == 0) {
        d.h_slot[0] = 0;
        d.root[turn] = {0, 0, 0ull};
    }
}

__global__ void __launch_bounds__(512)
train_begin_kernel(const TrainDesc *__restrict__ descs)
{
    Desc &d = FS_CONST(TrainDesc, descs)[blockIdx.x];
    begin_tree(d, 0);
    if (threadIdx.x == 0)
        d.root[1] = {0, 0, 0ull};
}

__device__ __forceinline__ int quantize(float g, float grad_scale)
{
    float t = g * grad_scale;
    t = fmaxf(t, -2147483520.0f);
    t = fminf(t, 2147483520.0f);
    return (int)rintf(t);
}

typedef int i32x4 __attribute__((ext_vector_type(4)));

// Cross-lane steps as DPP moves (register to register, no trip through the
// LDS crossbar as with __shfl): CTRL 0x110 + n = the lane n places down in its row of 16,
// 0x142 / 0x143 = last lane of the previous row / of the first two rows, for the rows named in
// ROW_MASK.  A lane without a source gets 0.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_i(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ long long dpp_ll(long long v)
{
    const int lo = dpp_i<CTRL, ROW_MASK>((int)v), hi = dpp_i<CTRL, ROW_MASK>((int)(v >> 32));
    return (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned long long)(unsigned)lo);
}

// Inclusive prefix sum over the 64 lanes: four doubling steps inside the rows of 16, then the
// total of row 0 (2) goes to row 1 (3), then the total of the first 32 lanes to the last 32.
__device__ __forceinline__ long long wave_prefix_ll(long long v)
{
    v += dpp_ll<0x111, 0xf>(v);
    v += dpp_ll<0x112, 0xf>(v);
    v += dpp_ll<0x114, 0xf>(v);
    v += dpp_ll<0x118, 0xf>(v);
    v += dpp_ll<0x142, 0xa>(v);
    v += dpp_ll<0x143, 0xc>(v);
    return v;
}

// The same as 32-bit adds whose operand comes through DPP; a lane without a source is not written.  (A DPP operand may
// not have been written by the last two instructions.)
__device__ __forceinline__ unsigned long long wave_prefix_u64(unsigned long long v)
{
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#define FS_PREFIX_STEP(how) \
    "v_add_co_u32_dpp %0, vcc, %0, %0 " how " bank_mask:0xf\n\t" \
    "v_addc_co_u32_dpp %1, vcc, %1, %1, vcc " how " bank_mask:0xf\n\t"
    asm("s_nop 1\n\t" FS_PREFIX_STEP("row_shr:1 row_mask:0xf") "s_nop 0\n\t" FS_PREFIX_STEP("row_shr:2 row_mask:0xf")
        "s_nop 0\n\t" FS_PREFIX_STEP("row_shr:4 row_mask:0xf") "s_nop 0\n\t" FS_PREFIX_STEP("row_shr:8 row_mask:0xf")
        "s_nop 0\n\t" FS_PREFIX_STEP("row_bcast:15 row_mask:0xa") "s_nop 0\n\t" FS_PREFIX_STEP("row_bcast:31 row_mask:0xc")
        "s_nop 1"
        : "+v"(lo), "+v"(hi)
        :
        : "vcc");
#undef FS_PREFIX_STEP
    return (unsigned long long)hi << 32 | lo;
}

__device__ __forceinline__ long long lane63_ll(long long v)
{
    const int lo = __builtin_amdgcn_readlane((int)v, 63), hi = __builtin_amdgcn_readlane((int)(v >> 32), 63);
    return (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned long long)(unsigned)lo);
}

// One thread per program.  `with_grad` = false only refreshes prog_pred.  A chain of latencies: rows are loaded sixteen
// at a time (the sum keeps their order) and the first sixteen are kept for their records; loaded again one by one, each
// behind the store of the record before, they were most of the launch.  One wavefront per workgroup spreads over the
// chip; of many programs four share the three atomics, which all go to the same addresses.  A round's launch: 4000 programs
// of 8.5 rows 6.5 -> 4.0 us, eight families of them 6.9 -> 5.2, 30 000 in one family 11.3 -> 6.3.
constexpr int kGradThreads = 64, kGradManyThreads = 256;
// Programs of a family from which on workgroups have four wavefronts: 8000 of 8.5 rows 4.6 us with one and 4.8 with four, of
// 1.5 rows 4.2 and 4.2, 12 000 5.4 and 5.1, 5.0 and 4.1, 16 000 6.2 and 5.6, 5.9 and 4.1, four families of 30 000 18.4 and 14.7; 4000
// 3.9 and 4.9, four families of them 4.4 and 5.4.
constexpr int kGradMany = 10000;
constexpr int kGradRows = 16;

// Bits of the sum over the wavefront.
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v)
{
    return (unsigned long long)lane63_ll((long long)wave_prefix_u64(v));
}

template <int THREADS>
__global__ void __launch_bounds__(THREADS)
train_grad_kernel(const TrainDesc *__restrict__ descs, float grad_scale, int with_grad, int turn)
{
    Desc &d = FS_CONST(TrainDesc, descs)[blockIdx.y];
    const int p = blockIdx.x * THREADS + threadIdx.x;
    long long G = 0, H = 0;
    unsigned long long A = 0;                        // |gradient| x rows: bounds every histogram sum
    if (p < d.n_programs) {
        auto preds = FS_GLOBAL(const float, d.row_pred);
        const int b = d.prog_off[p], e = d.prog_off[p + 1];
        const float target = with_grad ? d.target[p] : 0.0f;
        float first[kGradRows] = {}, s = 0.0f;
        in_runs<kGradRows>(b, e, [&](int r, int left) {
            float v[kGradRows];
#pragma unroll
            for (int i = 0; i < kGradRows; ++i)
                v[i] = preds[i < left ? r + i : e - 1];
#pragma unroll
            for (int i = 0; i < kGradRows; ++i) {
                s = i < left ? s + v[i] : s;
                first[i] = r == b ? v[i] : first[i];
            }
        });
        d.prog_pred[p] = s;
        if (with_grad) {
            const int q = quantize(s - target, grad_scale);
            const int len = e - b;
            auto recs = FS_GLOBAL(i32x4, d.rec[0]);
            in_runs<kGradRows>(b, e, [&](int r, int left) {
                if (r > b) {
#pragma unroll
                    for (int i = 0; i < kGradRows; ++i)
                        first[i] = preds[i < left ? r + i : e - 1];
                }
#pragma unroll
                for (int i = 0; i < kGradRows; ++i)
                    if (i < left)
                        recs[r + i] = (i32x4){r + i, q, len, __float_as_int(first[i])};
            });
            G = (long long)q * len;
            H = (long long)len * len;
            A = (unsigned long long)(G < 0 ? -G : G);
        }
    }
    if (!with_grad)
        return;
    // root totals: sums of the wavefronts, one atomic per workgroup
    constexpr int kWaves = THREADS / 64;
    unsigned long long sum[3] = {wave_sum_u64((unsigned long long)G), wave_sum_u64((unsigned long long)H), wave_sum_u64(A)};
    if (kWaves > 1) {
        __shared__ unsigned long long s_sum[kWaves][3];
        if ((threadIdx.x & 63) == 0)
            for (int k = 0; k < 3; ++k)
                s_sum[threadIdx.x >> 6][k] = sum[k];
        __syncthreads();
        for (int k = 0; k < 3; ++k) {
            sum[k] = 0;
            for (int w = 0; w < kWaves; ++w)
                sum[k] += s_sum[w][k];
        }
    }
    if (threadIdx.x == 0 && sum[1] != 0) {
        RootSums *sums = d.root + turn;
        atomicAdd((unsigned long long *)&sums->G, sum[0]);
        atomicAdd((unsigned long long *)&sums->H, sum[1]);
        atomicAdd(&sums->abs_q, sum[2]);
    }
}

// The node's own term of the gain, g*g/(H+lambda): the same for every cut of the node, so it is
// divided once per (node, feature) and not once per cut.
__device__ __forceinline__ double parent_term(long long G, long long H, double inv_scale, double lambda)
{
    const double g = (double)G * inv_scale;
    double t3 = g * g;
    t3 = t3 / ((double)H + lambda);
    return t3;
}

__device__ __forceinline__ double split_gain(long long GL, long long HL, long long G, long long H,
                                             double inv_scale, double lambda, double t3)
{
    const long long GR = G - GL, HR = H - HL;
    const double gl = (double)GL * inv_scale, gr = (double)GR * inv_scale;
    double t1 = gl * gl;
    t1 = t1 / ((double)HL + lambda);
    double t2 = gr * gr;
    t2 = t2 / ((double)HR + lambda);
    return (t1 + t2) - t3;
}

// One step of the arg-max over the lanes (largest gain, lowest cut on ties; cut 0 = nothing):
// the lane takes the other lane's pair if that is better.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ void best_step(double &best, int &best_cut)
{
    const long long bits = __double_as_longlong(best);
    const double og = __longlong_as_double(dpp_ll<CTRL, ROW_MASK>(bits));
    const int oc = dpp_i<CTRL, ROW_MASK>(best_cut);
    if (oc != 0 && (best_cut == 0 || og > best || (og == best && oc < best_cut))) {
        best = og;
        best_cut = oc;
    }
}

// The counted child of a split node: less curvature, or fewer rows where they are known; the left one on ties.
__device__ __forceinline__ int counts_left(long long l, long long r) { return l <= r ? 1 : 0; }

// Totals of a node; `turn` says which of the root's sums the round uses.  (No launch that calls this writes the totals
// of the level's nodes: with a uniform node they are scalar loads.)
__device__ __forceinline__ void node_sums(Desc &d, int node, int turn, long long &G, long long &H)
{
    if (node == 0) {
        G = *FS_CONST(long long, &d.root[turn].G);
        H = *FS_CONST(long long, &d.root[turn].H);
    } else {
        G = *FS_CONST(long long, d.h_G + node);
        H = *FS_CONST(long long, d.h_H + node);
    }
}

// Best cut of feature f for the open node `node`, by one wavefront: lane l holds bins 4l..4l+3
// (g, h; the feature's most frequent bin holds 0 and is rebuilt here from the node's totals)
// and forms the left sums of the cuts 4l+1..4l+4.  Lane 0 writes the result for
// `pair` = slot * F + f.
//
// A cut behind an empty bin splits the node exactly as the cut before it does: same gain, and
// coming later it never wins.  (A row's curvature is at least 1, so a bin is empty exactly when
// its H is 0.)  Deep in a tree a node holds fewer rows than a feature has bins and most cuts
// drop out this way; when at most 64 are left they are handed out one per lane through
// `scratch` (kCutScratchBytes of LDS that only this wavefront touches), so that the wavefront pays for one
// round of double-precision divisions instead of four.
constexpr int kCutScratchBytes = 64 * (8 + 8 + 4);

__device__ __forceinline__ void wave_best_cut(Desc &d, const Params &prm, int node, int turn, int f,
                                              int pair, int lane, long long (&g)[4], long long (&h)[4],
                                              unsigned char *scratch)
{
    long long G, H;
    node_sums(d, node, turn, G, H);
    const int hot = d.hot_bin[f];
    // inclusive prefix sums over the 256 bins, the hot bin still at 0
    const long long lane_g = g[0] + g[1] + g[2] + g[3], lane_h = h[0] + h[1] + h[2] + h[3];
    const long long pg = wave_prefix_ll(lane_g), ph = wave_prefix_ll(lane_h);
    // what the counted bins lack of the node's totals sits in the hot bin
    const long long hot_g = G - lane63_ll(pg), hot_h = H - lane63_ll(ph);
    long long before_g = pg - lane_g, before_h = ph - lane_h;
    if ((hot >> 2) < lane) {
        before_g += hot_g;
        before_h += hot_h;
    }
    if ((hot >> 2) == lane) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if ((hot & 3) == k) {
                g[k] = hot_g;
                h[k] = hot_h;
            }
    }
    bool filled[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        filled[k] = h[k] != 0;
#pragma unroll
    for (int k = 1; k < 4; ++k) {
        g[k] += g[k - 1];
        h[k] += h[k - 1];
    }
    const int m = d.cut_off[f + 1] - d.cut_off[f];
    const double t3 = parent_term(G, H, prm.inv_scale, prm.lambda);
    // cut 4l+k+1 (left = bins 0..4l+k) is worth evaluating if it is in range, follows a
    // non-empty bin and leaves enough curvature on both sides
    bool cand[4];
    unsigned long long vote[4];
    int n_cand = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const long long HL = before_h + h[k];
        cand[k] = 4 * lane + k + 1 <= m && filled[k] && HL >= prm.mcw && H - HL >= prm.mcw;
        vote[k] = __ballot(cand[k]);
        n_cand += __popcll(vote[k]);
    }
    int cut = 0;
    double gain = 0.0;
    long long bGL = 0, bHL = 0;
    if (n_cand <= 64) {
        // one candidate per lane (which lane takes which does not matter: ties are settled on
        // the cut number below)
        long long *s_GL = (long long *)scratch;
        long long *s_HL = s_GL + 64;
        int *s_cut = (int *)(s_HL + 64);
        const unsigned long long below = (1ull << lane) - 1ull;
        int first = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (cand[k]) {
                const int at = first + __popcll(vote[k] & below);
                s_GL[at] = before_g + g[k];
                s_HL[at] = before_h + h[k];
                s_cut[at] = 4 * lane + k + 1;
            }
            first += __popcll(vote[k]);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (lane < n_cand) {
            bGL = s_GL[lane];
            bHL = s_HL[lane];
            cut = s_cut[lane];
            gain = split_gain(bGL, bHL, G, H, prm.inv_scale, prm.lambda, t3);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();                         // the next search of this wavefront reuses the scratch
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (cand[k]) {
                const long long GL = before_g + g[k], HL = before_h + h[k];
                const double gn = split_gain(GL, HL, G, H, prm.inv_scale, prm.lambda, t3);
                if (cut == 0 || gn > gain) {                     // ascending cuts: first of equals stays
                    gain = gn;
                    cut = 4 * lane + k + 1;
                    bGL = GL;
                    bHL = HL;
                }
            }
        }
    }
    double best = gain;
    int best_cut = cut;
    // largest gain, lowest cut on ties: the same steps as the prefix sum leave the best of all
    // lanes in lane 63
    best_step<0x111, 0xf>(best, best_cut);
    best_step<0x112, 0xf>(best, best_cut);
    best_step<0x114, 0xf>(best, best_cut);
    best_step<0x118, 0xf>(best, best_cut);
    best_step<0x142, 0xa>(best, best_cut);
    best_step<0x143, 0xc>(best, best_cut);
    best_cut = __builtin_amdgcn_readlane(best_cut, 63);
    if (best_cut == 0) {
        if (lane == 0)
            d.best[pair].cut = 0;
    } else if (cut == best_cut) {                                // exactly one lane holds the winner
        d.best[pair] = {gain, cut, counts_left(bHL, H - bHL), bGL, bHL};
    }
}

// Largest of a value over the wavefront, by the steps of the prefix sum.
__device__ __forceinline__ float wave_max_f(float v)
{
#define FS_MAX_STEP(how) "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 " how " bank_mask:0xf\n\t"
    asm(FS_MAX_STEP("row_shr:1 row_mask:0xf") FS_MAX_STEP("row_shr:2 row_mask:0xf") FS_MAX_STEP("row_shr:4 row_mask:0xf")
        FS_MAX_STEP("row_shr:8 row_mask:0xf") FS_MAX_STEP("row_bcast:15 row_mask:0xa") FS_MAX_STEP("row_bcast:31 row_mask:0xc")
        "s_nop 1"
        : "+v"(v));
#undef FS_MAX_STEP
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// The same for packed bins (G * 2^hb + H, hb <= 31).  Bound by instruction issue where a level has many nodes (42 000
// searches of 164 features in 8 families: 25 us, 30 with the sums' steps and the nodes' values in vector code), by
// its chain of loads elsewhere (one family of 4000 programs: 5.9 us, 6.7 so), so:
//  - G and H go through one prefix sum, still packed.
//  - what the level's nodes are and hold comes by scalar loads.
//  - GL^2/(HL+lambda) + GR^2/(HR+lambda) is formed in float first, and only cuts within 2^-18 of
//    the largest are evaluated as the definition says, usually one.  The float value is within
//    10 * 2^-24 of the true one (G and GL times 2^hb are multiples of 2^hb below 2^63, and below
//    2^(31+2hb) since there are fewer than 2^hb rows: at most 53 bits, so their difference in double is
//    exact; G in units of 2^-hb is below 2^63 and its square is taken times the
//    reciprocal, so nothing overflows; a reciprocal that underflows leaves 0 for every cut, and
//    all are evaluated).  The gain itself is that sum minus a term that is the same for all cuts
//    and at most twice the sum, so a cut that wins after the rounding of double arithmetic is
//    within 2^-50 of the largest and never dropped.
__device__ __forceinline__ void wave_best_cut_packed(Desc &d, const Params &prm, int node, int turn,
                                                     int f, int pair, int lane, unsigned long long (&v)[4], int hb)
{
    long long G, H;
    node_sums(d, node, turn, G, H);
    const int hot = *FS_CONST(int32_t, d.hot_bin + f);
    const unsigned mask = (1u << hb) - 1u;
    const unsigned long long total = (unsigned long long)(G * ((long long)1 << hb) + H);
    const unsigned long long mine = v[0] + v[1] + v[2] + v[3];
    const unsigned long long incl = wave_prefix_u64(mine);
    // what the counted bins lack of the node's totals sits in the hot bin
    const unsigned long long rest = total - (unsigned long long)lane63_ll((long long)incl);
    unsigned long long before = incl - mine + ((hot >> 2) < lane ? rest : 0ull);
    const unsigned before_H = (unsigned)before & mask;
    const unsigned long long here = (hot >> 2) == lane ? rest : 0ull;
    switch (hot & 3) {
    case 0: v[0] += here; break;
    case 1: v[1] += here; break;
    case 2: v[2] += here; break;
    default: v[3] += here;
    }
    const int mcw = (int)min(prm.mcw, 0x7fffffffll), H_all = (int)H;
    const float lambda = (float)prm.lambda;
    const double G_all = (double)(long long)(total - (unsigned long long)H);
    // (Cuts behind the feature's last one leave no curvature on the right, and mcw is at least 1.)
    float t[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        before += v[k];
        v[k] = before;                                           // left sums of cut 4 * lane + k + 1
        const unsigned low = (unsigned)before;
        const int HL = (int)(low & mask), HR = H_all - HL;
        const double GL = __builtin_fma((double)(int)(before >> 32), 0x1p32, (double)(low & ~mask));   // times 2^hb
        const float gl = (float)GL, gr = (float)(G_all - GL);
        const float l = gl * __builtin_amdgcn_rcpf((float)HL + lambda), r = gr * __builtin_amdgcn_rcpf((float)HR + lambda);
        t[k] = HL >= mcw && HR >= mcw ? __builtin_fmaf(gl, l, gr * r) : -1.0f;
    }
    const float most = wave_max_f(fmaxf(fmaxf(t[0], t[1]), fmaxf(t[2], t[3])));
    const float least = most * (1.0f - 0x1p-18f);                // more than -1
    unsigned long long votes[4];
    int n_cand = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        votes[k] = __builtin_amdgcn_ballot_w64(!(t[k] < least));
        n_cand += __popcll(votes[k]);
    }
    if (n_cand > 1) {                                            // less those behind an empty bin
        n_cand = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            votes[k] &= __builtin_amdgcn_ballot_w64((((unsigned)v[k] & mask) != (k ? (unsigned)v[k ? k - 1 : 0] & mask : before_H)));
            n_cand += __popcll(votes[k]);
        }
    }
    if (n_cand == 0) {
        if (lane == 0)
            d.best[pair].cut = 0;
        return;
    }
    int cut = 0;
    double best = 0.0;
    long long bGL = 0, bHL = 0;
    const double t3 = node == 0 ? parent_term(G, H, prm.inv_scale, prm.lambda) : *FS_CONST(double, d.h_own + node);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (votes[k] == 0)
            continue;
        if (votes[k] >> lane & 1) {
            const long long HL = (long long)((unsigned)v[k] & mask);
            const long long GL = ((long long)v[k] - HL) >> hb;   // the difference is a multiple of 2^hb
            const double gn = split_gain(GL, HL, G, H, prm.inv_scale, prm.lambda, t3);
            if (cut == 0 || gn > best) {                         // ascending cuts: first of equals stays
                best = gn;
                cut = 4 * lane + k + 1;
                bGL = GL;
                bHL = HL;
            }
        }
    }
    const double gain = best;
    int best_cut = cut;
    if (n_cand > 1) {
        // largest gain, lowest cut on ties: the same steps as the prefix sum leave the best of all
        // lanes in lane 63
        best_step<0x111, 0xf>(best, best_cut);
        best_step<0x112, 0xf>(best, best_cut);
        best_step<0x114, 0xf>(best, best_cut);
        best_step<0x118, 0xf>(best, best_cut);
        best_step<0x142, 0xa>(best, best_cut);
        best_step<0x143, 0xc>(best, best_cut);
        best_cut = __builtin_amdgcn_readlane(best_cut, 63);
    }
    if (cut != 0 && cut == best_cut)                             // exactly one lane holds the winner
        d.best[pair] = {gain, cut, counts_left(bHL, H - bHL), bGL, bHL};
}

// Histograms of one level.
//
// Of two siblings only one is counted, the one with fewer rows or, before they are known, less curvature; the
// other is the parent's histogram minus it.  All sums are integer sums, so that is exact.  A work item is up to 2^shift
// rows; a workgroup takes one item and sixteen features, walks the item's records and gathers each row's
// bins, 16 bytes at a time.
//
// Two ways.  After train_move_kernel the items are the counted nodes' own records (ALL).  In train_grow_kernel
// they are the parents', moved by other workgroups of the same launch: every workgroup decides its parent
// and adds the rows that go to the counted child (a byte gathered from the split feature's column says
// which).  That saves a launch of dependent loads a level, 5 to 6 us, and visits twice the rows with half of
// the lanes idle: a round of depth 6 of 2500 / 8500 / 25 500 / 51 000 / 60 500 rows takes 83 / 94 / 108 /
// 129 / 153 us grown and 99 / 108 / 118 / 129 / 150 moved first (kGrowRows), 255 000 rows 240 and 203.  (Compacting
// the rows through a queue in LDS instead of leaving lanes idle: 117 us at 25 500 rows, 223 at 255 000.)
//
// A node of a single item leaves its histogram in its place of `hist`; the items of larger ones
// write their part and train_split_kernel adds the parts up.  (Parts are stored and not added atomically:
// nothing has to be cleared, and the memory-side atomics of eight XCDs are slower than the extra
// read.)  The cut search is a kernel of its own: in here it held the row loop to 6 wavefronts a
// SIMD and a node's sixteen features to eight wavefronts; depth 6, 25 500 rows: 15 us for the
// histograms and cuts of 8 nodes.
//
// Bound by the LDS: 64-bit adds of 64 lanes on 32 bank pairs at random take about 20 clocks a wavefront.
//
// Two forms of a bin.  Packed: one 64-bit word G * 2^hb + H, fed by one atomic per (row, feature);
// hb bits hold any curvature sum (the host knows rows x longest program) and the rest holds G as
// long as the sum of |gradient| over the trainer's rows, which train_grad_kernel leaves in `root`,
// stays below 2^(63-hb).  Wide: G and H in 64 bits each, always safe, eight features at a time in
// the same LDS; H has a plane of its own in the buffers.  Every kernel of a round decides alike.
constexpr int kHistThreads = 512;
constexpr int64_t kGrowRows = 49152;    // of a batch
static_assert(kBins * 8 >= kCutScratchBytes, "room for the cut search's scratch");

__device__ __forceinline__ bool is_packed(Desc &d, int turn, int hb)
{
    return hb > 0 && *FS_CONST(unsigned long long, &d.root[turn].abs_q) < (1ull << (63 - hb));
}

// Records of a node (heap index) and which of its pieces of 2^shift rows a workgroup takes.
struct Piece {
    int node;
    int first, count;         // records of the whole node
    int piece;
};

__device__ __forceinline__ int wave_prefix_i(int v)
{
    v += dpp_i<0x111, 0xf>(v);
    v += dpp_i<0x112, 0xf>(v);
    v += dpp_i<0x114, 0xf>(v);
    v += dpp_i<0x118, 0xf>(v);
    v += dpp_i<0x142, 0xa>(v);
    v += dpp_i<0x143, 0xc>(v);
    return v;
}

__device__ __forceinline__ int pieces_of(int count, int shift)
{
    return (int)(((int64_t)count + (1ll << shift) - 1) >> shift);
}

// Piece number `index` of the level's nodes (every wavefront finds it for itself: one 16-byte load per
// parent and a scan).
__device__ __forceinline__ bool find_piece(Desc &d, int level, int shift, int index, int lane, Piece &it)
{
    if (level == 0) {
        it = {0, 0, d.n_rows, index};
        return index < pieces_of(d.n_rows, shift);
    }
    constexpr int kMost = (1 << (FS_TRAIN_MAX_DEPTH - 2)) / 64;   // parents per lane
    const int n_parents = 1 << (level - 1);
    const int per = n_parents > 64 ? n_parents / 64 : 1;
    int4 s[kMost];
    int sum = 0;
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
        const int p = lane * per + i;
        s[i] = i < per && p < n_parents ? d.seg[n_parents - 1 + p] : make_int4(0, 0, 0, 0);
        sum += pieces_of(s[i].x, shift) + pieces_of(s[i].y, shift);
    }
    const int incl = wave_prefix_i(sum);
    const unsigned long long past = __ballot(incl > index);
    if (past == 0)
        return false;
    const int owner = __builtin_amdgcn_readfirstlane(__ffsll((long long)past) - 1);
    int rest = index - (incl - sum);
    Piece mine = {-1, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < kMost; ++i)
#pragma unroll
        for (int right = 0; right < 2; ++right) {
            const int count = right ? s[i].y : s[i].x, n = pieces_of(count, shift);
            if (mine.node < 0 && rest < n)
                mine = {2 * (n_parents - 1 + lane * per + i) + 1 + right, s[i].z + (right ? s[i].x : 0), count, rest};
            rest -= n;
        }
    it.node = __builtin_amdgcn_readlane(mine.node, owner);
    it.first = __builtin_amdgcn_readlane(mine.first, owner);
    it.count = __builtin_amdgcn_readlane(mine.count, owner);
    it.piece = __builtin_amdgcn_readlane(mine.piece, owner);
    return true;
}

// The same over the counted children of the level.
__device__ __forceinline__ bool find_counted(Desc &d, int level, int shift, int index, int lane, Piece &it)
{
    if (level == 0) {
        it = {0, 0, d.n_rows, index};
        return index < pieces_of(d.n_rows, shift);
    }
    constexpr int kMost = (1 << (FS_TRAIN_MAX_DEPTH - 2)) / 64;   // parents per lane
    const int n_parents = 1 << (level - 1);
    const int per = n_parents > 64 ? n_parents / 64 : 1;
    int first[kMost], count[kMost], left[kMost], sum = 0;
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
        const int p = lane * per + i, node = n_parents - 1 + (i < per && p < n_parents ? p : 0);
        const int4 s = d.seg[node];
        left[i] = counts_left(s.x, s.y);
        first[i] = left[i] ? s.z : s.z + s.x;
        count[i] = i < per && p < n_parents ? (left[i] ? s.x : s.y) : 0;
        sum += pieces_of(count[i], shift);
    }
    const int incl = wave_prefix_i(sum);
    const unsigned long long past = __ballot(incl > index);
    if (past == 0)
        return false;
    const int owner = __builtin_amdgcn_readfirstlane(__ffsll((long long)past) - 1);
    int rest = index - (incl - sum);
    Piece mine = {-1, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
        const int n = pieces_of(count[i], shift);
        if (mine.node < 0 && rest < n)
            mine = {2 * (n_parents - 1 + lane * per + i) + 2 - left[i], first[i], count[i], rest};
        rest -= n;
    }
    it.node = __builtin_amdgcn_readlane(mine.node, owner);
    it.first = __builtin_amdgcn_readlane(mine.first, owner);
    it.count = __builtin_amdgcn_readlane(mine.count, owner);
    it.piece = __builtin_amdgcn_readlane(mine.piece, owner);
    return true;
}

// Where the parts of a node of several items start in `part`.  Two nodes never overlap: one of
// c > 2^shift rows has at most ceil(c / 2^shift) <= floor(2c / 2^shift) parts.
__device__ __forceinline__ int64_t part_slot(int first, int shift)
{
    return (2 * (int64_t)first) >> shift;
}

template <bool PACKED>
struct Bins4 {                // four consecutive bins of a lane
    unsigned long long a[4], b[PACKED ? 1 : 4];
    __device__ __forceinline__ void load(const unsigned long long *p, int64_t plane)
    {
        typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
        const u64x2 u = ((const u64x2 *)p)[0], v = ((const u64x2 *)p)[1];
        a[0] = u.x, a[1] = u.y, a[2] = v.x, a[3] = v.y;
        if (!PACKED) {
            const u64x2 x = ((const u64x2 *)(p + plane))[0], y = ((const u64x2 *)(p + plane))[1];
            b[0] = x.x, b[PACKED ? 0 : 1] = x.y, b[PACKED ? 0 : 2] = y.x, b[PACKED ? 0 : 3] = y.y;
        }
    }
    __device__ __forceinline__ void store(unsigned long long *p, int64_t plane) const
    {
        typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
        ((u64x2 *)p)[0] = (u64x2){a[0], a[1]};
        ((u64x2 *)p)[1] = (u64x2){a[2], a[3]};
        if (!PACKED) {
            ((u64x2 *)(p + plane))[0] = (u64x2){b[0], b[PACKED ? 0 : 1]};
            ((u64x2 *)(p + plane))[1] = (u64x2){b[PACKED ? 0 : 2], b[PACKED ? 0 : 3]};
        }
    }
    __device__ __forceinline__ void add(const Bins4 &o, bool minus)
    {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            a[k] = minus ? o.a[k] - a[k] : a[k] + o.a[k];
        if (!PACKED)
#pragma unroll
            for (int k = 0; k < (PACKED ? 1 : 4); ++k)
                b[k] = minus ? o.b[k] - b[k] : b[k] + o.b[k];
    }
};

// Words of a node's histogram of feature f; at the root and for counted children a place of their own,
// for the other child its parent's.  `pair`: number of the parent within its level.
__device__ __forceinline__ int64_t hist_at(Desc &d, int level, int pair, int which, int f)
{
    const int n_pairs = level > 0 ? 1 << (level - 1) : 0;
    const int slot = level == 0 ? 0 : which ? *FS_CONST(int32_t, d.h_slot + n_pairs - 1 + pair) : n_pairs + pair;
    return ((int64_t)slot * d.n_features + f) * kBins;
}

// Two siblings: the counted one and the other (-1 at the root).
struct Pair {
    int small, large;
    int pair;                 // number of the parent within its level
    int first, count;         // records that were dealt out in pieces
};

// Cuts of one child: `which` = 0 the counted node, 1 its sibling; `own`: the counted node's bins.
template <bool PACKED>
__device__ __forceinline__ void search_child(Desc &d, const Params &prm, int level, int turn, const Pair &it,
                                             int which, bool store, int f, int lane, Bins4<PACKED> &own, int hb,
                                             unsigned char *scratch)
{
    const int node = which ? it.large : it.small;
    unsigned long long *place = d.hist + hist_at(d, level, it.pair, which, f) + 4 * lane;
    if (which) {
        Bins4<PACKED> parent;
        parent.load(place, d.hist_plane);
        own.add(parent, true);
    }
    if (store && level + 1 < prm.max_depth)
        own.store(place, d.hist_plane);
    const int pair = (node - ((1 << level) - 1)) * d.n_features + f;
    if constexpr (PACKED) {
        unsigned long long v[4] = {own.a[0], own.a[1], own.a[2], own.a[3]};
        wave_best_cut_packed(d, prm, node, turn, f, pair, lane, v, hb);
    } else {
        long long g[4] = {(long long)own.a[0], (long long)own.a[1], (long long)own.a[2], (long long)own.a[3]};
        long long h[4] = {(long long)own.b[0], (long long)own.b[1], (long long)own.b[2], (long long)own.b[3]};
        wave_best_cut(d, prm, node, turn, f, pair, lane, g, h, scratch);
    }
}

// What the next level needs of two siblings: their places in `hist` and their segments, nothing moved yet.
__device__ __forceinline__ void open_children(Desc &d, int level, const Pair &it)
{
    const int parent = (1 << (level - 1)) - 1 + it.pair, left = 2 * parent + 1;
    const int4 s = d.seg[parent];
    d.h_slot[it.small] = (1 << (level - 1)) + it.pair;
    d.h_slot[it.large] = d.h_slot[parent];
    d.seg[left] = make_int4(0, 0, s.z, s.z + s.x);
    d.seg[left + 1] = make_int4(0, 0, s.z + s.x, s.w);
}

// One node's outcome, the same in every workgroup that works on it.
struct Decision {
    int split;                // else a leaf
    int feature, cut;
    int count_left;           // the left child is the counted one
    float left, right;        // values of the children that become leaves; of the node itself in `left`
};

__device__ __forceinline__ float leaf_value(long long G, long long H, const Params &prm)
{
    const double g = (double)G * prm.inv_scale;
    return (float)(-prm.eta * g / ((double)H + prm.lambda));
}

// Decides node `node` of the level, by one wavefront (lanes over the features): largest gain, lowest
// feature on ties.  Everybody waits for this, so it reads and reduces no more than that.
__device__ __forceinline__ Decision wave_decide(Desc &d, int level, const Params &prm, int node, int lane)
{
    double gain = 0.0;
    int feature = -1, cut = 0;                                   // cut * 2 + count_left
    if (level < prm.max_depth) {
        auto best = FS_GLOBAL(const i32x4, d.best + (int64_t)(node - ((1 << level) - 1)) * d.n_features);
        constexpr int kPerLane = 3;                              // loads at a time: this is a chain of latencies
        for (int f0 = lane; f0 < d.n_features; f0 += 64 * kPerLane) {
            i32x4 o[kPerLane];                                   // a record's first half
#pragma unroll
            for (int i = 0; i < kPerLane; ++i)
                o[i] = best[2 * min(f0 + 64 * i, d.n_features - 1)];
#pragma unroll
            for (int i = 0; i < kPerLane; ++i) {                 // ascending: first of equals stays
                const int f = f0 + 64 * i;
                const double g = __longlong_as_double((long long)((unsigned long long)(unsigned)o[i].y << 32 | (unsigned)o[i].x));
                if (f < d.n_features && o[i].z != 0 && (feature < 0 || g > gain)) {
                    gain = g;
                    feature = f;
                    cut = 2 * o[i].z + o[i].w;
                }
            }
        }
    }
    const double mine = gain;
    int id = feature + 1;                                        // as in the cut search: 0 = nothing
    best_step<0x111, 0xf>(gain, id);
    best_step<0x112, 0xf>(gain, id);
    best_step<0x114, 0xf>(gain, id);
    best_step<0x118, 0xf>(gain, id);
    best_step<0x142, 0xa>(gain, id);
    best_step<0x143, 0xc>(gain, id);
    id = __builtin_amdgcn_readlane(id, 63);
    const unsigned long long who = __ballot(feature + 1 == id && mine > prm.min_gain);
    Decision r = {};
    if (id != 0 && who != 0) {
        cut = __builtin_amdgcn_readlane(cut, __ffsll((long long)who) - 1);
        r.split = 1;
        r.feature = id - 1;
        r.cut = cut >> 1;
        r.count_left = cut & 1;
    }
    return r;
}

// Values of the leaves that a decision makes.
__device__ __forceinline__ void leaf_values(Desc &d, int level, int turn, const Params &prm, int node,
                                            Decision &r)
{
    if (r.split && level + 1 < prm.max_depth)
        return;
    long long G, H;
    node_sums(d, node, turn, G, H);
    if (!r.split) {
        r.left = leaf_value(G, H, prm);
        return;
    }
    const Best b = d.best[(int64_t)(node - ((1 << level) - 1)) * d.n_features + r.feature];
    r.left = leaf_value(b.GL, b.HL, prm);
    r.right = leaf_value(G - b.GL, H - b.HL, prm);
}

// What later launches read of a decided node (one lane of one of its workgroups).
__device__ __forceinline__ void note_decision(Desc &d, int level, int turn, const Params &prm, int node,
                                              const Decision &r)
{
    if (!r.split) {
        d.decision[node] = make_int4(kLeaf, 0, 0, __float_as_int(r.left));
        return;
    }
    const int lc = 2 * node + 1, rc = lc + 1;
    d.decision[node] = make_int4(kInternal, r.feature, 0, __float_as_int(d.cuts[d.cut_off[r.feature] + r.cut - 1]));
    if (level + 1 >= prm.max_depth) {
        d.h_val[lc] = r.left;
        d.h_val[rc] = r.right;
        return;
    }
    long long G, H;
    node_sums(d, node, turn, G, H);
    const Best b = d.best[(int64_t)(node - ((1 << level) - 1)) * d.n_features + r.feature];
    d.h_G[lc] = b.GL;
    d.h_H[lc] = b.HL;
    d.h_G[rc] = G - b.GL;
    d.h_H[rc] = H - b.HL;
    d.h_own[lc] = parent_term(b.GL, b.HL, prm.inv_scale, prm.lambda);
    d.h_own[rc] = parent_term(G - b.GL, H - b.HL, prm.inv_scale, prm.lambda);
}

// Heap -> flat arrays, appended to the model; then the heap is the next tree's (one workgroup of
// kHistThreads).  Ids are local to the tree in breadth-first order, which is the heap's order.  `ids`: LDS.
__device__ __forceinline__ void emit_tree(Desc &d, int max_depth, int turn, int *ids)
{
    constexpr int kPer = (kHeapNodes + kHistThreads) / kHistThreads;
    __shared__ int s_sum[kHistThreads / 64];
    const int n_trees = d.counters[1], base = d.counters[2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_heap = (2 << max_depth) - 1;
    int4 c[kPer];
    int sum = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int i = threadIdx.x * kPer + k;
        const bool deepest = i >= (1 << max_depth) - 1;
        c[k] = make_int4(kAbsent, 0, 0, 0);
        if (i < n_heap) {
            c[k] = d.decision[deepest && max_depth > 0 ? (i - 1) >> 1 : i];
            const float v = d.h_val[i];
            if (deepest && max_depth > 0)
                c[k] = make_int4(c[k].x == kInternal ? kLeaf : kAbsent, 0, 0, __float_as_int(v));
        }
        sum += c[k].x != kAbsent;
    }
    const int incl = wave_prefix_i(sum);
    if (lane == 63)
        s_sum[wave] = incl;
    __syncthreads();
    int id = incl - sum, total = 0;
    for (int w = 0; w < kHistThreads / 64; ++w) {
        id += w < wave ? s_sum[w] : 0;
        total += s_sum[w];
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int i = threadIdx.x * kPer + k;
        if (i < n_heap)
            ids[i] = id;
        id += c[k].x != kAbsent;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int i = threadIdx.x * kPer + k;
        if (c[k].x == kAbsent)
            continue;
        const int at = base + ids[i];
        const bool inner = c[k].x == kInternal;
        d.m_feat[at] = inner ? c[k].y : -1;
        d.m_thr[at] = inner ? __int_as_float(c[k].w) : 0.0f;
        d.m_left[at] = inner ? ids[2 * i + 1] : -1;
        d.m_right[at] = inner ? ids[2 * i + 2] : -1;
        d.m_val[at] = inner ? 0.0f : __int_as_float(c[k].w);
    }
    if (threadIdx.x == 0) {
        d.counters[1] = n_trees + 1;
        d.counters[2] = base + total;
        d.m_tree_off[n_trees + 1] = base + total;
    }
    begin_tree(d, turn);
}

__global__ void __launch_bounds__(kHistThreads)
train_emit_kernel(const TrainDesc *__restrict__ descs, int max_depth, int turn)
{
    __shared__ int ids[kHeapNodes];
    emit_tree(FS_CONST(TrainDesc, descs)[blockIdx.x], max_depth, turn, ids);
}

struct HistLds {
    unsigned long long bins[kHistWords];
    Decision dec;
};

// The histogram of a counted node of level `child` (number `pair` of its parents): features f0 + base .. + NF of the
// piece's rows, ALL of them (the piece is the node's) or those that go to it (the piece is its parent's, which
// is decided here, while the first rows and their bins are on their way).
template <bool PACKED, bool ALL>
__device__ __forceinline__ void hist_run(Desc &d, HistLds &s, const Piece &it, int child, int pair, int shift,
                                         int group, int base, int hb, const Params &prm)
{
    constexpr int NF = PACKED ? kHistFeats : kHistFeats / 2;
    constexpr int NW = NF / 4;
    const int f0 = group * kHistFeats + base;
    const int nf = min(NF, d.n_features - f0);
    unsigned long long *lds = s.bins;
    const int n = min(it.count - (int)((int64_t)it.piece << shift), 1 << shift);
    auto recs = FS_GLOBAL(const i32x4, d.rec[ALL ? child & 1 : (child - 1) & 1] + it.first + ((int64_t)it.piece << shift));
    typedef uint32_t words __attribute__((ext_vector_type(NW)));
    auto bins = FS_GLOBAL(const uint8_t, d.bins + f0);
    const int64_t row_bytes = d.row_bytes;
    typedef __attribute__((address_space(1))) const words *words_at;
    // (the records of a group are read in order, its bins gathered: the loads of the next step are
    // issued before the atomics of this one)
    int i = threadIdx.x;
    i32x4 r = {}, r_next = {};
    words w = {};
    if (i < n) {
        r = recs[i];
        r_next = recs[min(i + kHistThreads, n - 1)];
    }
    for (int j = threadIdx.x; j < kHistWords; j += kHistThreads)
        lds[j] = 0ull;
    auto hots = FS_CONST(int32_t, d.hot_bin + f0);
    int hot[NF];
#pragma unroll
    for (int k = 0; k < NF; ++k) {
        hot[k] = hots[min(k, nf - 1)];                           // (no branch: sixteen scalar loads at once)
        hot[k] = k < nf ? hot[k] : 256;                          // 256: no bin, nothing is skipped
    }
    if (i < n)
        w = *(words_at)(bins + r.x * row_bytes);
    if (!ALL && threadIdx.x < 64) {
        const Decision mine = wave_decide(d, child - 1, prm, it.node, threadIdx.x);
        if (threadIdx.x == 0)
            s.dec = mine;
    }
    __syncthreads();
    int cut = 0, count_left = 0;
    auto col = FS_GLOBAL(const uint8_t, d.cols);
    int b = 0;
    if (!ALL) {
        if (!s.dec.split)
            return;
        cut = s.dec.cut;
        count_left = s.dec.count_left;
        col = FS_GLOBAL(const uint8_t, d.cols + s.dec.feature * d.r_pad);
        b = i < n ? col[(uint32_t)r.x] : 0;
    }
    for (; i < n; i += kHistThreads) {
        const words w_next = *(words_at)(bins + r_next.x * row_bytes);
        const int b_next = ALL ? 0 : col[(uint32_t)r_next.x];
        const i32x4 r_after = recs[min(i + 2 * kHistThreads, n - 1)];
        if (ALL || (b < cut) == (count_left != 0)) {
            const unsigned long long both = (unsigned long long)((long long)r.y * ((long long)1 << hb) + (long long)r.z);
#pragma unroll
            for (int k = 0; k < NF; ++k) {
                if ((k & 3) == 0 && k >= nf)
                    break;
                const int bin = (w[k >> 2] >> (8 * (k & 3))) & 255;
                if (bin != hot[k]) {
                    atomicAdd(&lds[k * kBins + bin], PACKED ? both : (unsigned long long)(long long)r.y);
                    if (!PACKED)
                        atomicAdd(&lds[kHistWords / 2 + k * kBins + bin], (unsigned long long)r.z);
                }
            }
        }
        r = r_next;
        w = w_next;
        b = b_next;
        r_next = r_after;
    }
    __syncthreads();
    const bool whole = it.count <= 1 << shift;
    const int64_t plane = whole ? d.hist_plane : d.part_plane;
    unsigned long long *out =
        whole ? d.hist + hist_at(d, child, pair, 0, f0)
              : d.part + ((part_slot(it.first, shift) + it.piece) * d.n_features + f0) * kBins;
    for (int j = 2 * threadIdx.x; j < nf * kBins; j += 2 * kHistThreads) {
        *(ulonglong2 *)(out + j) = *(ulonglong2 *)(lds + j);
        if (!PACKED)
            *(ulonglong2 *)(out + plane + j) = *(ulonglong2 *)(lds + kHistWords / 2 + j);
    }
    __syncthreads();                                             // LDS may be reused by the next run
}

template <bool ALL>
__device__ __forceinline__ void hist_both(Desc &d, HistLds &s, const Piece &it, int child, int pair, int turn,
                                          int shift, int group, int hb, const Params &prm)
{
    if (is_packed(d, turn, hb)) {
        hist_run<true, ALL>(d, s, it, child, pair, shift, group, 0, hb, prm);
    } else {
        hist_run<false, ALL>(d, s, it, child, pair, shift, group, 0, 0, prm);
        if (group * kHistFeats + kHistFeats / 2 < d.n_features)
            hist_run<false, ALL>(d, s, it, child, pair, shift, group, kHistFeats / 2, 0, prm);
    }
}

// Histograms of the level's counted nodes, whose records are in place (of its LDS hist_run uses the bins only).
// Behind them, in layer `emit`, one workgroup per trainer puts the tree of the round before into the model.
__global__ void __launch_bounds__(kHistThreads)
train_hist_kernel(const TrainDesc *__restrict__ descs, int level, int turn, int shift, int hb, int emit, int max_depth)
{
    __shared__ __align__(16) unsigned long long lds[kHistWords];
    HistLds &s = *(HistLds *)lds;
    Desc &d = FS_CONST(TrainDesc, descs)[blockIdx.y];
    if ((int)blockIdx.z == emit) {
        if (blockIdx.x == 0)
            emit_tree(d, max_depth, turn ^ 1, (int *)lds);
        return;
    }
    Piece it;
    const int item = xcd_piece(blockIdx.x, blockIdx.y, blockIdx.z), group = (int)blockIdx.x >> 3;
    if (group * kHistFeats >= d.n_features || !find_counted(d, level, shift, item, threadIdx.x & 63, it))
        return;
    hist_both<true>(d, s, it, level, level ? ((it.node - 1) >> 1) - ((1 << (level - 1)) - 1) : 0, turn, shift, group, hb,
                    Params());
}

// Records of a node that is split move to its children's segments in the other buffer: the left child's
// fill the node's segment from its front, the right one's from its back (the order inside a segment is
// free: all sums over rows are integer sums).  Rows of leaves take the leaf's value.
// A workgroup takes kMoveRows rows of one node and counts them up with one atomic; bound by its chain of
// three barriers and six loads.  Two rows a thread: one takes 212 us for a round of depth 6 of 255 000 rows (as
// many atomics again on one address near the root), two 203, four 201, and 218 / 217 / 220 for depth 8
// of 102 000.  On the last level nothing moves.
constexpr int kMovePer = 2;
constexpr int kMoveRows = kMovePer * kHistThreads;
constexpr int kMoveShift = 10;
static_assert(kMoveRows == 1 << kMoveShift, "rows of a moving workgroup");

template <bool LAST>
__device__ __forceinline__ void move_rows(Desc &d, Decision &s_dec, const Piece &it, int level, int turn,
                                          const Params &prm)
{
    __shared__ int s_left[kHistThreads / 64], s_right[kHistThreads / 64];
    __shared__ unsigned long long s_base;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = min(it.count - it.piece * kMoveRows, kMoveRows);
    auto recs = FS_GLOBAL(const i32x4, d.rec[level & 1] + it.first + it.piece * kMoveRows);
    i32x4 r[kMovePer];
#pragma unroll
    for (int k = 0; k < kMovePer; ++k)
        r[k] = recs[min((int)threadIdx.x + k * kHistThreads, n - 1)];
    if (wave == 0) {
        Decision mine = wave_decide(d, level, prm, it.node, lane);
        leaf_values(d, level, turn, prm, it.node, mine);
        if (lane == 0)
            s_dec = mine;
    }
    __syncthreads();
    const Decision dec = s_dec;
    if (it.piece == 0 && threadIdx.x == kHistThreads - 1)
        note_decision(d, level, turn, prm, it.node, dec);
    if (!dec.split || LAST) {
        int b[kMovePer];
#pragma unroll
        for (int k = 0; k < kMovePer; ++k)
            b[k] = dec.split ? d.cols[dec.feature * d.r_pad + r[k].x] : 0;
#pragma unroll
        for (int k = 0; k < kMovePer; ++k)
            if ((int)threadIdx.x + k * kHistThreads < n)
                d.row_pred[r[k].x] = __int_as_float(r[k].w) + (!dec.split || b[k] < dec.cut ? dec.left : dec.right);
        return;
    }
    int b[kMovePer];
    unsigned long long lm[kMovePer], rm[kMovePer];
#pragma unroll
    for (int k = 0; k < kMovePer; ++k)
        b[k] = d.cols[dec.feature * d.r_pad + r[k].x];
    int wl = 0, wr = 0;
#pragma unroll
    for (int k = 0; k < kMovePer; ++k) {
        const bool in = (int)threadIdx.x + k * kHistThreads < n;
        lm[k] = __ballot(in && b[k] < dec.cut);
        rm[k] = __ballot(in && !(b[k] < dec.cut));
        wl += __popcll(lm[k]);
        wr += __popcll(rm[k]);
    }
    if (lane == 0) {
        s_left[wave] = wl;
        s_right[wave] = wr;
    }
    __syncthreads();
    int l = 0, rt = 0, l_all = 0, r_all = 0;
#pragma unroll
    for (int w = 0; w < kHistThreads / 64; ++w) {
        l += w < wave ? s_left[w] : 0;
        rt += w < wave ? s_right[w] : 0;
        l_all += s_left[w];
        r_all += s_right[w];
    }
    if (threadIdx.x == 0)
        s_base = atomicAdd((unsigned long long *)&d.seg[it.node],
                           (unsigned long long)(unsigned)l_all | (unsigned long long)(unsigned)r_all << 32);
    __syncthreads();
    const unsigned long long start = s_base, below = (1ull << lane) - 1ull;
    l += it.first + (int)(unsigned)start;
    rt += (int)(start >> 32);
    auto out = FS_GLOBAL(i32x4, d.rec[(level + 1) & 1]);
#pragma unroll
    for (int k = 0; k < kMovePer; ++k) {
        if ((int)threadIdx.x + k * kHistThreads < n)
            out[b[k] < dec.cut ? l + __popcll(lm[k] & below) : it.first + it.count - 1 - (rt + __popcll(rm[k] & below))] = r[k];
        l += __popcll(lm[k]);
        rt += __popcll(rm[k]);
    }
}

// One level: decides its nodes, moves their records, counts the smaller children.
// The first `layers` of the grid move.
__global__ void __launch_bounds__(kHistThreads)
train_grow_kernel(const TrainDesc *__restrict__ descs, int level, int turn, int shift, int hb, int layers, int movers,
                  Params prm)
{
    __shared__ __align__(16) HistLds s;
    const int lane = threadIdx.x & 63;
    Piece it;
    Desc &d = FS_CONST(TrainDesc, descs)[blockIdx.y];
    if ((int)blockIdx.z < layers) {
        const int index = (int)(blockIdx.z * gridDim.x + blockIdx.x);
        if (index < movers && find_piece(d, level, kMoveShift, index, lane, it))
            move_rows<false>(d, s.dec, it, level, turn, prm);
        return;
    }
    const int item = xcd_piece(blockIdx.x, blockIdx.y, blockIdx.z - layers), group = (int)blockIdx.x >> 3;
    if (group * kHistFeats >= d.n_features || !find_piece(d, level, shift, item, lane, it))
        return;
    hist_both<false>(d, s, it, level + 1, it.node - ((1 << level) - 1), turn, shift, group, hb, prm);
}

// The first half of a level by itself, where train_hist_kernel is to count the moved records.
__global__ void __launch_bounds__(kHistThreads)
train_move_kernel(const TrainDesc *__restrict__ descs, int level, int turn, Params prm)
{
    __shared__ Decision dec;
    Desc &d = FS_CONST(TrainDesc, descs)[blockIdx.y];
    Piece it;
    if (find_piece(d, level, kMoveShift, blockIdx.x, threadIdx.x & 63, it))
        move_rows<false>(d, dec, it, level, turn, prm);
}

// The last level: decides its nodes, rows take the values of the leaves.  blockIdx = (workgroup, trainer)
__global__ void __launch_bounds__(kHistThreads)
train_finish_kernel(const TrainDesc *__restrict__ descs, int level, int turn, Params prm)
{
    __shared__ Decision dec;
    Desc &d = FS_CONST(TrainDesc, descs)[blockIdx.y];
    Piece it;
    if (find_piece(d, level, kMoveShift, blockIdx.x, threadIdx.x & 63, it))
        move_rows<true>(d, dec, it, level, turn, prm);
}

// One workgroup per (counted node, feature): the wavefronts add up the node's parts if it has several,
// then one searches the node's cuts and another its sibling's, whose histogram takes the parent's place.
// Two wavefronts; four where the launch has so few workgroups, of nodes near the root with many parts each, that
// the adding up is a latency: a round of 65 000 rows of depth 6 takes 164.8 us against 166.4, of 255 000 239.6
// against 242.0.  In batches they only hold others up: eight families of 30 000 rows 299.7 against 295.7, five of
// 25 000 to 100 000 268.5 against 266.3.
constexpr int kSplitWaves = 4;
constexpr int kSplitWideNodes = 4;

template <bool PACKED>
__device__ __forceinline__ void split_run(Desc &d, const Params &prm, unsigned long long *lds,
                                          const Pair &it, int level, int turn, int shift, int f, int hb)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    const int children = level > 0 ? 2 : 1;
    const int pieces = pieces_of(it.count, shift);
    Bins4<PACKED> own = {};
    if (pieces > 1) {
        const unsigned long long *part = d.part + (part_slot(it.first, shift) * d.n_features + f) * kBins + 4 * lane;
        const int64_t stride = (int64_t)d.n_features * kBins;
#pragma unroll 4
        for (int j = wave; j < pieces; j += waves) {
            Bins4<PACKED> one;
            one.load(part + j * stride, d.part_plane);
            own.add(one, false);
        }
        own.store(lds + wave * kBins + 4 * lane, waves * kBins);
        __syncthreads();
        own = {};
        for (int j = 0; j < waves; ++j) {
            Bins4<PACKED> one;
            one.load(lds + j * kBins + 4 * lane, waves * kBins);
            own.add(one, false);
        }
        __syncthreads();                                         // the sums' LDS is the search's scratch now
        if (wave >= children)
            return;
    } else {
        if (wave >= children)
            return;
        own.load(d.hist + hist_at(d, level, it.pair, 0, f) + 4 * lane, d.hist_plane);
    }
    search_child<PACKED>(d, prm, level, turn, it, wave, wave || pieces > 1, f, lane, own, hb,
                         (unsigned char *)(lds + wave * kBins));
    if (f == 0 && wave == 0 && lane == 0 && level > 0 && level + 1 < prm.max_depth)
        open_children(d, level, it);
}

__global__ void __launch_bounds__(64 * kSplitWaves, 6)
train_split_kernel(const TrainDesc *__restrict__ descs, int level, int turn, int shift, int hb, int grown, Params prm)
{
    extern __shared__ __align__(16) unsigned long long lds[];
    Desc &d = FS_CONST(TrainDesc, descs)[blockIdx.z];
    const int f = blockIdx.x, pair = blockIdx.y;
    if (f >= d.n_features)
        return;
    Pair it = {0, -1, 0, 0, d.n_rows};
    if (level > 0) {
        const int parent = (1 << (level - 1)) - 1 + pair, left = 2 * parent + 1;
        const i32x4 s = *FS_CONST(i32x4, d.seg + parent);
        if (s.x == 0)                                            // not split
            return;
        const bool count_left = grown ? counts_left(*FS_CONST(long long, d.h_H + left), *FS_CONST(long long, d.h_H + left + 1))
                                      : counts_left(s.x, s.y);
        it = {count_left ? left : left + 1, count_left ? left + 1 : left, pair, s.z, s.x + s.y};
        if (!grown) {                                            // the pieces are the counted node's
            it.first = count_left ? s.z : s.z + s.x;
            it.count = count_left ? s.x : s.y;
        }
    }
    if (is_packed(d, turn, hb))
        split_run<true>(d, prm, lds, it, level, turn, shift, f, hb);
    else
        split_run<false>(d, prm, lds, it, level, turn, shift, f, 0);
}

}  // namespace fs

// ---- host side ----------------------------------------------------------------------------

namespace fs {

// A call's work on the device: done where the event is.
struct Work {
    hipEvent_t done = nullptr;
    ~Work()
    {
        if (done)
            (void)hipEventDestroy(done);
    }
};

}  // namespace fs

struct fs_trainer {
    fs::TrainDesc h;          // host copy of the descriptor (device pointers inside)
    int device;
    int max_depth, max_trees;
    int trees_enqueued;
    int max_len;              // rows of the longest program
    void *memory;             // everything the descriptor points to
    size_t memory_bytes;
    std::shared_ptr<fs::Work> last;   // of the calls that work in the memory; none: nothing is at work
    bool untracked;           // something may be that `last` does not tell
};

namespace fs {

static std::mutex g_train_mu;
struct BatchBuf {
    TrainDesc *d_desc = nullptr;
    TrainDesc *h_desc = nullptr;   // pinned
    int cap = 0;
    void *work = nullptr;          // histograms of the batch in work: room for any batch of `alive`
    size_t work_bytes = 0;
    std::vector<const fs_trainer *> alive;   // without any `work` is kept up to kKeptWork
    struct Block { void *p; size_t bytes; std::shared_ptr<Work> last; };
    std::vector<Block> kept;       // memory of destroyed trainers, for the next
    size_t kept_bytes = 0;
    void *staging[4] = {};         // pinned memory that no call uses
    size_t needed = 0, needed_before = 0;    // of `work`, since there was no trainer; and until then
    hipEvent_t copied = nullptr;
    bool pending = false;
    std::shared_ptr<Work> last;    // of fs_train_boost and fs_trainer_predictions, each of which waits for it first
};
static BatchBuf *const g_batch = new BatchBuf[16];   // never freed: trainers may outlive static objects

// The histograms' buffer stays between the trainers of one tuning step and the next up to this size:
// mapping and freeing it for every retraining took 0.7 to 1.3 ms of 6.5 to 17 (what a batch needs beyond
// goes with the device's last trainer, all of it where device memory runs out for something else).
constexpr size_t kKeptWork = (size_t)512 << 20;

// Memory of destroyed trainers stays for the next ones up to this: allocating and freeing it cost 210 us a trainer
// (eight retrained families: 1.7 of 15 ms).  Room for two jobs of the largest kind: a model of 255 000 rows of 164
// features takes 101 MB, eight of 34 000 rows 108; and for one of more families than the paper's networks have (38).
// Every allocation of the library takes it back before it fails.
constexpr size_t kKeptBlocks = (size_t)256 << 20;
constexpr size_t kMostKept = 64;

// Small host arrays go through pinned memory that kernels read and write: a plain copy waits 14 to 36 us.
constexpr size_t kStagingBytes = (size_t)512 << 10;

// Frees the kept blocks (g_train_mu held).
static bool free_kept(BatchBuf &b)
{
    const bool any = !b.kept.empty();
    for (const BatchBuf::Block &k : b.kept)
        (void)hipFree(k.p);
    b.kept.clear();
    b.kept_bytes = 0;
    return any;
}

// Frees the kept blocks and the histograms' buffer of a device without trainers (g_train_mu held).
static bool give_back(BatchBuf &b)
{
    const bool any = free_kept(b);
    if (!b.alive.empty() || !b.work)
        return any;
    (void)hipFree(b.work);
    b.work = nullptr;
    b.work_bytes = 0;
    return true;
}

// device_malloc for who holds g_train_mu.
static hipError_t malloc_or_give_back(BatchBuf &b, void **p, size_t bytes)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory && give_back(b)) {
        (void)hipGetLastError();
        e = hipMalloc(p, bytes);
    }
    return e;
}

// Keeps a destroyed trainer's memory, or frees it, which waits for the device.  `last` may still be at work in it:
// take_block's caller waits for that.
static void keep_block(BatchBuf &b, void *p, size_t bytes, const std::shared_ptr<Work> &last)
{
    if (bytes > kKeptBlocks) {
        (void)hipFree(p);
        return;
    }
    while (!b.kept.empty() && (b.kept_bytes + bytes > kKeptBlocks || b.kept.size() >= kMostKept)) {   // the oldest first
        (void)hipFree(b.kept.front().p);
        b.kept_bytes -= b.kept.front().bytes;
        b.kept.erase(b.kept.begin());
    }
    try {
        b.kept.push_back({p, bytes, last});
        b.kept_bytes += bytes;
    } catch (const std::bad_alloc &) {
        (void)hipFree(p);
    }
}

// A kept block for `bytes`, not more than twice as large; null if there is none.
static void *take_block(int device, size_t bytes, size_t *size, std::shared_ptr<Work> *last)
{
    if (device < 0 || device >= 16)
        return nullptr;
    std::lock_guard<std::mutex> lock(g_train_mu);
    BatchBuf &b = g_batch[device];
    size_t best = b.kept.size();
    for (size_t i = 0; i < b.kept.size(); ++i)
        if (b.kept[i].bytes >= bytes && b.kept[i].bytes / 2 <= bytes && (best == b.kept.size() || b.kept[i].bytes < b.kept[best].bytes))
            best = i;
    if (best == b.kept.size())
        return nullptr;
    void *p = b.kept[best].p;
    *size = b.kept[best].bytes;
    *last = b.kept[best].last;
    b.kept_bytes -= *size;
    b.kept.erase(b.kept.begin() + (long)best);
    return p;
}

// kStagingBytes of pinned memory for a call that waits for what it starts, or null.
class Staging {
public:
    Staging(int device, size_t bytes) : device_(device)
    {
        if (device < 0 || device >= 16 || bytes > kStagingBytes)
            return;
        {
            std::lock_guard<std::mutex> lock(g_train_mu);
            for (void *&s : g_batch[device].staging)
                if (s) {
                    p = s;
                    s = nullptr;
                    return;
                }
        }
        if (hipHostMalloc(&p, kStagingBytes, hipHostMallocDefault) != hipSuccess) {
            p = nullptr;
            (void)hipGetLastError();
        }
    }
    ~Staging()
    {
        if (!p)
            return;
        {
            std::lock_guard<std::mutex> lock(g_train_mu);
            for (void *&s : g_batch[device_].staging)
                if (!s) {
                    s = p;
                    return;
                }
        }
        (void)hipHostFree(p);
    }
    Staging(const Staging &) = delete;
    Staging &operator=(const Staging &) = delete;
    void *p = nullptr;

private:
    int device_;
};

bool give_back_training_memory(int device)
{
    if (device < 0 || device >= 16)
        return false;
    std::lock_guard<std::mutex> lock(g_train_mu);
    return give_back(g_batch[device]);
}

// The arrays of a trainer lie in one device allocation: noted first, placed when all are known.
struct Arena {
    struct Part { void **out; size_t at; };
    Part part[48];
    int n = 0;
    size_t bytes = 0;
    template <class T>
    void add(T **out, size_t count)
    {
        part[n++] = {(void **)out, bytes};
        bytes += ((count ? count : 1) * sizeof(T) + 255) & ~(size_t)255;
    }
    int place(void **base, size_t *size, int device)
    {
        std::shared_ptr<Work> last;
        *base = take_block(device, bytes, size, &last);
        if (last) {                                              // not for whatever else the device does
            const hipError_t e = hipEventSynchronize(last->done);
            if (e != hipSuccess) {
                (void)hipFree(*base);
                *base = nullptr;
                return fail_hip(e, "waiting for a destroyed trainer");
            }
        }
        const hipError_t e = *base ? hipSuccess : hipMalloc(base, *size = bytes);
        if (e != hipSuccess) {
            *base = nullptr;
            (void)hipGetLastError();                             // not the next launch's error
            return e == hipErrorOutOfMemory ? fail(FS_ENOMEM, "hipMalloc of %zu bytes failed", bytes)
                                            : fail_hip(e, "hipMalloc");
        }
        for (int i = 0; i < n; ++i)
            *part[i].out = (char *)*base + part[i].at;
        return FS_OK;
    }
};

static int check_launch(const char *what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return fail_hip(e, what);
    return FS_OK;
}

// ---- the histograms' buffer --------------------------------------------------------------------
// Histograms live for one fs_train_boost only, and training calls on one device are ordered by the
// caller, as its descriptors need already: all trainers share a buffer of the device (fresh memory of
// 20 MB for each of eight trainers took 5 ms of a job's retraining).  fs_trainer_create
// grows it to what any batch of the trainers alive may need, so that fs_train_boost
// neither allocates nor waits.  A batch that needs more than kMostWork is trained in parts, one after the other.
constexpr size_t kMostWork = (size_t)16 << 30;

static size_t most_work()
{
    const int mb = tune(FS_TUNE_TRAIN_WORK_MB);                  // test override
    return mb >= 1 ? (size_t)mb << 20 : kMostWork;
}

// Bits that hold any curvature sum of a batch (rows x longest program bounds it).  The packed form of the
// histograms needs room for the gradient sums beside them; beyond 31 bits the wide form is
// taken right away (0).
static int packed_bits(int max_len, int max_rows)
{
    int hb = 1;
    while (hb < 63 && ((long long)1 << hb) <= (long long)max_len * (long long)max_rows)
        ++hb;
    return hb > 31 || tune(FS_TUNE_TRAIN_PACKED) == 0 ? 0 : hb;  // override: wide form only
}

// Planes of a trainer's histograms: one where the packed form can never give way to the wide one, as no
// gradient exceeds 31 bits (quantize).
static int hist_planes(const fs_trainer *t, int hb)
{
    return hb > 0 && hb <= 32 && t->h.n_rows <= (int64_t)1 << (32 - hb) ? 1 : 2;
}

// Words of the histograms that trees of `depth` levels keep, and of the parts of nodes of several items, in
// a plane; returns the bytes of all planes.
static size_t hist_bytes(const fs_trainer *t, int depth, int shift, int hb, size_t *hist, size_t *part)
{
    const size_t row = (size_t)t->h.n_features * kBins;
    const int64_t rows = t->h.n_rows;
    *hist = (depth > 0 ? (size_t)1 << (depth - 1) : 1) * row;
    *part = rows >> shift ? ((size_t)((2 * rows) >> shift) + 1) * row : 0;
    return (*hist + *part) * hist_planes(t, hb) * sizeof(unsigned long long);
}

// What a batch of any of these trainers takes at most.  With items of 2^shift rows the batch's parts are 2 R >> shift
// and one more per trainer; shift is kChunkShiftMin or such that R are at most kMostGroups items of all features.
static size_t any_batch_bytes(const std::vector<const fs_trainer *> &trainers)
{
    int max_len = 0, max_rows = 0;
    for (const fs_trainer *t : trainers) {
        max_len = std::max(max_len, t->max_len);
        max_rows = std::max(max_rows, t->h.n_rows);
    }
    const int hb = packed_bits(max_len, max_rows);
    // words of the parts of that many items: groups of features are whole ones at most
    const size_t most = (size_t)2 * kMostGroups * kHistWords;
    size_t hists = 0, parts = 0, largest_row = 0, largest_plane = 0, single = 0;
    for (const fs_trainer *t : trainers) {
        size_t hist, part;
        (void)hist_bytes(t, t->max_depth, kChunkShiftMin, hb, &hist, &part);
        const size_t words = (size_t)t->h.n_features * kBins, plane = sizeof(unsigned long long) * hist_planes(t, hb);
        hists += hist * plane;
        parts += part / words;
        largest_row = std::max(largest_row, words * plane);
        largest_plane = std::max(largest_plane, plane);
        single = std::max(single, (hist + std::min(part, most + words)) * plane);
    }
    const size_t all = hists + std::min(parts * largest_row, most * largest_plane + trainers.size() * largest_row);
    return std::max(single, std::min(all, most_work()));
}

// The buffer grows to `bytes`, or `wish` if that is to be had (g_train_mu held).  Where neither is, it is
// what it was.
static int grow_work(BatchBuf &b, size_t bytes, size_t wish)
{
    FS_HIP(hipDeviceSynchronize());                              // earlier batches may still be at work in it
    const size_t had = b.work_bytes;
    if (b.work)
        (void)hipFree(b.work);
    b.work = nullptr;
    b.work_bytes = 0;
    hipError_t e = hipErrorOutOfMemory;
    for (const size_t size : {wish, bytes, had}) {
        if (size == 0)
            continue;
        const hipError_t err = malloc_or_give_back(b, &b.work, size);
        if (err == hipSuccess) {
            b.work_bytes = size;
            break;
        }
        e = err;
        b.work = nullptr;
        (void)hipGetLastError();                                 // not the next launch's error
    }
    if (b.work_bytes >= bytes)
        return FS_OK;
    return e == hipErrorOutOfMemory ? fail(FS_ENOMEM, "hipMalloc of %zu bytes for histograms failed", bytes)
                                    : fail_hip(e, "hipMalloc");
}

// Counts the trainer among its device's and makes room for it.
static int reserve_work(const fs_trainer *t)
{
    if (t->device < 0 || t->device >= 16)
        return FS_OK;                                            // fs_train_boost turns it down
    std::lock_guard<std::mutex> lock(g_train_mu);
    BatchBuf &b = g_batch[t->device];
    try {
        b.alive.push_back(t);
    } catch (const std::bad_alloc &) {
        return fail(FS_ENOMEM, "out of host memory");
    }
    const size_t need = any_batch_bytes(b.alive);
    b.needed = std::max(b.needed, need);
    if (b.work_bytes >= need)
        return FS_OK;
    // The trainers of a job are created one after the other: at once what the job before needed, else in
    // steps.  (Eight trainers of depth 10, 1.5 GB: 4 ms in steps, 0.3 at once.)
    return grow_work(b, need, std::max({need, b.needed_before, std::min(2 * b.work_bytes, b.work_bytes + kKeptWork)}));
}

}  // namespace fs

using namespace fs;

extern "C" void fs_trainer_destroy(fs_trainer *t)
{
    if (!t)
        return;
    const bool keeps = !t->untracked && t->device >= 0 && t->device < 16;
    if (t->memory && !keeps)
        (void)hipFree(t->memory);
    if (t->device >= 0 && t->device < 16) {
        std::lock_guard<std::mutex> lock(g_train_mu);
        BatchBuf &b = g_batch[t->device];
        if (t->memory && keeps)
            keep_block(b, t->memory, t->memory_bytes, t->last);
        const auto it = std::find(b.alive.begin(), b.alive.end(), t);
        if (it != b.alive.end()) {
            b.alive.erase(it);
            if (b.alive.empty()) {
                b.needed_before = b.needed;
                b.needed = 0;
                if (b.work_bytes > kKeptWork) {
                    (void)hipFree(b.work);
                    b.work = nullptr;
                    b.work_bytes = 0;
                }
            }
        }
    }
    delete t;
}

extern "C" int fs_trainer_create(fs_trainer **out, int32_t n_features, const float *features,
                                 int32_t layout, int64_t n_rows, const int32_t *prog_off,
                                 int32_t n_programs, const float *target, const int32_t *cut_off,
                                 const float *cuts, float bias, int32_t max_depth, int32_t max_trees,
                                 void *stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (!out)
        return fail(FS_EINVAL, "fs_trainer_create: out is NULL");
    *out = nullptr;
    if (n_features < 1 || n_features > FS_MAX_FEATURES)
        return fail(FS_EINVAL, "fs_trainer_create: n_features=%d outside 1..%d", n_features, FS_MAX_FEATURES);
    if (n_rows < 1 || n_rows >= (int64_t)1 << 31 || n_programs < 1)
        return fail(FS_EINVAL, "fs_trainer_create: n_rows=%lld, n_programs=%d must be >= 1",
                    (long long)n_rows, n_programs);
    if (!features || !prog_off || !target || !cut_off || (!cuts && cut_off[n_features] > 0))
        return fail(FS_EINVAL, "fs_trainer_create: NULL argument");
    if (layout != FS_ROWMAJOR && layout != FS_COLBLOCK64)
        return fail(FS_EINVAL, "fs_trainer_create: unknown layout %d", layout);
    if (max_depth < 0 || max_depth > FS_TRAIN_MAX_DEPTH)
        return fail(FS_EUNSUPPORTED, "fs_trainer_create: max_depth=%d outside 0..%d", max_depth,
                    FS_TRAIN_MAX_DEPTH);
    if (max_trees < 1)
        return fail(FS_EINVAL, "fs_trainer_create: max_trees=%d must be >= 1", max_trees);
    if (cut_off[0] != 0)
        return fail(FS_EINVAL, "fs_trainer_create: cut_off[0] must be 0");
    for (int f = 0; f < n_features; ++f) {
        const int m = cut_off[f + 1] - cut_off[f];
        if (m < 0 || m > FS_TRAIN_MAX_CUTS)
            return fail(m < 0 ? FS_EINVAL : FS_EUNSUPPORTED,
                        "fs_trainer_create: feature %d has %d cuts (0..%d allowed)", f, m, FS_TRAIN_MAX_CUTS);
        for (int j = 0; j < m; ++j) {
            const float c = cuts[cut_off[f] + j];
            if (c != c || (j > 0 && !(cuts[cut_off[f] + j - 1] < c)))
                return fail(FS_EINVAL, "fs_trainer_create: cuts of feature %d are not ascending and distinct", f);
        }
    }
    fs_trainer *t = new (std::nothrow) fs_trainer();
    if (!t)
        return fail(FS_ENOMEM, "out of host memory");
    int rc = FS_OK;
    hipError_t e = hipGetDevice(&t->device);
    if (e != hipSuccess) {
        delete t;
        return fail_hip(e, "hipGetDevice");
    }
    t->max_depth = max_depth;
    t->max_trees = max_trees;
    t->trees_enqueued = 0;
    t->untracked = true;                                         // until this call's work is done
    TrainDesc &h = t->h;
    h.n_features = n_features;
    h.n_rows = (int32_t)n_rows;
    h.n_programs = n_programs;
    h.bias = bias;
    h.r_pad = (n_rows + 255) & ~(int64_t)255;
    const int n_cuts = cut_off[n_features];
    const int hist_slots = max_depth > 0 ? 1 << (max_depth - 1) : 1;
    const int64_t node_cap = (int64_t)max_trees * ((1 << (max_depth + 1)) - 1);
    uint8_t *bins = nullptr, *cols = nullptr;
    int32_t *d_prog_off = nullptr, *d_cut_off = nullptr;
    float *d_target = nullptr, *d_cuts = nullptr;
    int32_t *d_hot = nullptr;
    uint32_t *d_count = nullptr;
    int32_t *d_longest = nullptr;
    const int clear_blocks = (int)std::min<int64_t>(1024, std::max<int64_t>(32, n_rows / 1024));
    Arena arena;
    // whole pieces of a row, and of a 64-byte sector from four pieces on
    h.row_bytes = (n_features + kHistFeats - 1) / kHistFeats * kHistFeats;
    h.row_bytes = h.row_bytes > 2 * kHistFeats ? (h.row_bytes + 63) & ~63 : h.row_bytes;
    arena.add(&bins, (size_t)n_rows * (size_t)h.row_bytes);
    arena.add(&cols, (size_t)h.r_pad * (size_t)n_features);
    arena.add(&d_prog_off, (size_t)n_programs + 1);
    arena.add(&d_target, (size_t)n_programs);
    arena.add(&d_cut_off, (size_t)n_features + 1 + (size_t)n_cuts);   // the cuts lie behind
    arena.add(&d_hot, (size_t)n_features);
    arena.add(&d_count, (size_t)n_features * kBins);
    arena.add(&d_longest, (size_t)clear_blocks);
    arena.add(&h.row_pred, (size_t)n_rows);
    arena.add(&h.prog_pred, (size_t)n_programs);
    arena.add(&h.rec[0], (size_t)n_rows);
    arena.add(&h.rec[1], (size_t)n_rows);
    arena.add(&h.seg, (size_t)kHeapNodes);
    arena.add(&h.h_slot, (size_t)kHeapNodes);
    arena.add(&h.h_own, (size_t)kHeapNodes);
    arena.add(&h.h_val, (size_t)kHeapNodes);
    arena.add(&h.h_G, (size_t)kHeapNodes);
    arena.add(&h.h_H, (size_t)kHeapNodes);
    arena.add(&h.best, (size_t)hist_slots * n_features);
    arena.add(&h.decision, (size_t)kHeapNodes);
    arena.add(&h.counters, (size_t)4);
    arena.add(&h.root, (size_t)2);
    arena.add(&h.m_tree_off, (size_t)max_trees + 1);
    arena.add(&h.m_feat, (size_t)node_cap);
    arena.add(&h.m_left, (size_t)node_cap);
    arena.add(&h.m_right, (size_t)node_cap);
    arena.add(&h.m_thr, (size_t)node_cap);
    arena.add(&h.m_val, (size_t)node_cap);
    rc = arena.place(&t->memory, &t->memory_bytes, t->device);
    if (rc == FS_ENOMEM && give_back_training_memory(t->device))
        rc = arena.place(&t->memory, &t->memory_bytes, t->device);
    if (rc != FS_OK) {
        fs_trainer_destroy(t);
        return rc;
    }
    d_cuts = (float *)(d_cut_off + n_features + 1);
    h.bins = bins;
    h.cols = cols;
    h.prog_off = d_prog_off;
    h.target = d_target;
    h.cut_off = d_cut_off;
    h.cuts = d_cuts;
    h.hot_bin = d_hot;
    e = hipMemcpyAsync(d_prog_off, prog_off, sizeof(int32_t) * ((size_t)n_programs + 1),
                       hipMemcpyDeviceToDevice, stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(d_target, target, sizeof(float) * (size_t)n_programs,
                           hipMemcpyDeviceToDevice, stream);
    // the small host arrays, staged [longest program, cut_off, cuts] or, if too long for that, in one plain copy
    const size_t head = (size_t)n_features + 1, n_words = head + (size_t)n_cuts;
    const Staging staging(t->device, sizeof(int32_t) * (n_words + 1));
    int32_t *const staged = (int32_t *)staging.p;
    if (e == hipSuccess) {
        std::unique_ptr<int32_t[]> both(staged ? nullptr : new (std::nothrow) int32_t[n_words]);
        int32_t *const words = staged ? staged + 1 : both.get();
        if (!words) {
            fs_trainer_destroy(t);
            return fail(FS_ENOMEM, "out of host memory");
        }
        memcpy(words, cut_off, sizeof(int32_t) * head);
        if (n_cuts > 0)
            memcpy(words + head, cuts, sizeof(float) * (size_t)n_cuts);
        if (!staged)
            e = hipMemcpy(d_cut_off, words, sizeof(int32_t) * n_words, hipMemcpyHostToDevice);
    }
    if (e != hipSuccess) {
        fs_trainer_destroy(t);
        return fail_hip(e, "fs_trainer_create: copies");
    }
    hipLaunchKernelGGL(train_clear_kernel, dim3((unsigned)clear_blocks), dim3(kBins), 0, stream,
                       (const int32_t *)(staged ? staged + 1 : nullptr), (int)n_words, d_cut_off, d_count, n_features * kBins,
                       h.counters, h.m_tree_off, h.row_pred, (int64_t)n_rows, bias, (const int32_t *)d_prog_off, n_programs,
                       d_longest);
    hipLaunchKernelGGL(train_bin_kernel,
                       dim3((unsigned)((n_rows + 2047) / 2048 * 8 * ((n_features + kHistFeats - 1) / kHistFeats))),
                       dim3(256), 0, stream, features, layout, n_features, (int)n_rows, h.r_pad,
                       (const int32_t *)d_cut_off, (const float *)d_cuts, bins, h.row_bytes, cols);
    hipLaunchKernelGGL(train_count_kernel,
                       dim3((unsigned)((n_rows + kCountRows - 1) / kCountRows), (unsigned)n_features), dim3(256),
                       0, stream, (const uint8_t *)cols, (int)n_rows, h.r_pad, d_count);
    hipLaunchKernelGGL(train_hot_bin_kernel, dim3((unsigned)n_features + 1), dim3(kBins), 0, stream,
                       (const uint32_t *)d_count, n_features, d_hot, (const int32_t *)d_longest, clear_blocks, h.counters + 3,
                       staged);
    rc = check_launch("trainer set-up kernels launch");
    e = hipStreamSynchronize(stream);                            // (whatever has been launched reads the staging memory)
    t->untracked = e != hipSuccess;
    if (rc == FS_OK) {
        if (staged)
            t->max_len = staged[0];
        else if (e == hipSuccess)
            e = hipMemcpy(&t->max_len, h.counters + 3, sizeof(int32_t), hipMemcpyDeviceToHost);
        if (e != hipSuccess)
            rc = fail_hip(e, "fs_trainer_create: reading the longest program");
    }
    if (rc == FS_OK)
        rc = reserve_work(t);
    if (rc != FS_OK) {
        fs_trainer_destroy(t);
        return rc;
    }
    *out = t;
    return FS_OK;
}

// Work that trainers' memory, the descriptors and the histograms' buffer are in, between begin_work and end_work
// (g_train_mu held): behind that of the call before, on whichever stream, and noted for the next call and for who
// takes a trainer's memory over.  (One event for all trainers of a call; on one stream the wait costs nothing.)
// Not while the stream is captured: the work runs with the graph, and the trainers' memory is not kept.
static bool captured(hipStream_t stream)
{
    hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &s) == hipSuccess)
        return s != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

static int begin_work(BatchBuf &b, hipStream_t stream)
{
    if (b.last && !captured(stream))
        FS_HIP(hipStreamWaitEvent(stream, b.last->done, 0));
    return FS_OK;
}

static void end_work(BatchBuf &b, fs_trainer *const *trainers, int n, hipStream_t stream)
{
    std::shared_ptr<Work> work;
    try {
        work = std::make_shared<Work>();
    } catch (const std::bad_alloc &) {
    }
    const bool noted = work && !captured(stream) &&
                       hipEventCreateWithFlags(&work->done, hipEventDisableTiming) == hipSuccess &&
                       hipEventRecord(work->done, stream) == hipSuccess;
    for (int i = 0; i < n; ++i) {
        if (noted)
            trainers[i]->last = work;
        else
            trainers[i]->untracked = true;
    }
    if (noted)
        b.last = work;
    else
        (void)hipGetLastError();                                 // not the next launch's error
}

// `most`: programs of the largest of `n` trainers.
static void launch_grad(const TrainDesc *d, int most, unsigned n, float grad_scale, int with_grad, int turn, hipStream_t stream)
{
    const int threads = most > kGradMany ? kGradManyThreads : kGradThreads;
    const dim3 grid((unsigned)(((int64_t)most + threads - 1) / threads), n);
    if (most > kGradMany)
        hipLaunchKernelGGL(train_grad_kernel<kGradManyThreads>, grid, dim3(threads), 0, stream, d, grad_scale, with_grad, turn);
    else
        hipLaunchKernelGGL(train_grad_kernel<kGradThreads>, grid, dim3(threads), 0, stream, d, grad_scale, with_grad, turn);
}

// Uploads descriptors; returns the device array.
static int upload_batch(int n, const fs_trainer *const *trainers, hipStream_t stream, const TrainDesc **d_out)
{
    int dev = 0;
    FS_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 16)
        return fail(FS_EUNSUPPORTED, "device ordinal %d not supported", dev);
    BatchBuf &b = g_batch[dev];
    if (!b.copied)
        FS_HIP(hipEventCreateWithFlags(&b.copied, hipEventDisableTiming));
    if (b.pending) {
        FS_HIP(hipEventSynchronize(b.copied));     // the previous upload has left the staging buffer
        b.pending = false;
    }
    if (b.cap < n) {
        // earlier batches may still be read by kernels in flight
        FS_HIP(hipDeviceSynchronize());
        if (b.d_desc)
            FS_HIP(hipFree(b.d_desc));
        if (b.h_desc)
            FS_HIP(hipHostFree(b.h_desc));
        b.d_desc = b.h_desc = nullptr;
        b.cap = 0;
        const int cap = n < 16 ? 16 : 2 * n;
        FS_HIP(malloc_or_give_back(b, (void **)&b.d_desc, sizeof(TrainDesc) * (size_t)cap));
        FS_HIP(hipHostMalloc((void **)&b.h_desc, sizeof(TrainDesc) * (size_t)cap, hipHostMallocDefault));
        b.cap = cap;
    }
    for (int i = 0; i < n; ++i)
        b.h_desc[i] = trainers[i]->h;
    FS_HIP(hipMemcpyAsync(b.d_desc, b.h_desc, sizeof(TrainDesc) * (size_t)n, hipMemcpyHostToDevice, stream));
    FS_HIP(hipEventRecord(b.copied, stream));
    b.pending = true;
    *d_out = b.d_desc;
    return FS_OK;
}

static int check_batch(const char *who, int n, fs_trainer *const *trainers)
{
    if (n < 0)
        return fail(FS_EINVAL, "%s: n_trainers %d is negative", who, n);
    if (n > 0 && !trainers)
        return fail(FS_EINVAL, "%s: trainers is NULL", who);
    int dev = 0;
    FS_HIP(hipGetDevice(&dev));
    for (int i = 0; i < n; ++i) {
        if (!trainers[i])
            return fail(FS_EINVAL, "%s: trainer %d is NULL", who, i);
        if (trainers[i]->device != dev)
            return fail(FS_EINVAL, "%s: trainer %d lives on device %d, current is %d", who, i,
                        trainers[i]->device, dev);
        for (int j = 0; j < i; ++j)
            if (trainers[j] == trainers[i])
                return fail(FS_EINVAL, "%s: trainer %d appears twice in the batch", who, i);
    }
    return FS_OK;
}

namespace {

// Trainers [first, first + n) of a call, trained side by side.
struct Part {
    int first, n;
    int shift, hb;                   // rows of a histogram workgroup (log2); packed_bits
    bool grown;                      // the levels' records are moved and counted by one launch
    int max_rows, max_prog, max_feat;
    size_t bytes;                    // of histograms
};

Part make_part(const fs_trainer *const *trainers, int first, int n, int depth)
{
    Part pt = {first, n, kChunkShiftMin, 0, false, 0, 0, 0, 0};
    int max_len = 0;
    int64_t total_rows = 0;
    for (int i = first; i < first + n; ++i) {
        const fs_trainer *t = trainers[i];
        total_rows += t->h.n_rows;
        pt.max_rows = std::max(pt.max_rows, t->h.n_rows);
        pt.max_prog = std::max(pt.max_prog, t->h.n_programs);
        pt.max_feat = std::max(pt.max_feat, t->h.n_features);
        max_len = std::max(max_len, t->max_len);
    }
    // A histogram workgroup takes up to 2^shift rows of a node.
    const int64_t groups = (pt.max_feat + kHistFeats - 1) / kHistFeats;
    if (total_rows > kChunkSmallRows)
        ++pt.shift;
    pt.grown = total_rows <= kGrowRows;
    while (pt.shift < 30 && total_rows * groups > (int64_t)kMostGroups << pt.shift)
        ++pt.shift;
    const int v = tune(FS_TUNE_TRAIN_SLAB_ROWS);                 // test / tuning override
    if (v >= 64 && v <= 65536)
        for (pt.shift = 6; (1 << pt.shift) < v;)
            ++pt.shift;
    while (((int64_t)pt.max_rows >> pt.shift) + (1 << FS_TRAIN_MAX_DEPTH) > kMostPieces)
        ++pt.shift;
    pt.hb = packed_bits(max_len, pt.max_rows);
    size_t hist, part;
    for (int i = first; i < first + n; ++i)
        pt.bytes += hist_bytes(trainers[i], depth, pt.shift, pt.hb, &hist, &part);
    return pt;
}

// Enqueues the rounds of a part whose descriptors are at d.
int train_part(const TrainDesc *d, const Part &pt, int n_rounds, const Params &prm, hipStream_t stream)
{
    const unsigned nt = (unsigned)pt.n;
    const unsigned groups = (unsigned)((pt.max_feat + kHistFeats - 1) / kHistFeats);
    const int max_rows = pt.max_rows, shift = pt.shift, hb = pt.hb;
    const bool grown = pt.grown;
    prof_start(kKernTrainOther, stream);
    hipLaunchKernelGGL(train_begin_kernel, dim3(nt), dim3(512), 0, stream, d);
    prof_stop(stream);
    for (int round = 0; round < n_rounds; ++round) {
        const int turn = round & 1;
        prof_start(kKernTrainOther, stream);
        launch_grad(d, pt.max_prog, nt, prm.grad_scale, 1, turn, stream);
        prof_stop(stream);
        for (int level = 0; level < prm.max_depth; ++level) {    // histograms and cuts of the level's nodes
            const int64_t parents = level ? (int64_t)1 << (level - 1) : 1;
            // at most this many pieces of 2^s rows of so many nodes of r rows in all
            auto most = [&](int64_t r, int s) { return std::max<int64_t>(1, std::min<int64_t>(r, (r >> s) + parents)); };
            if (level && !grown) {
                prof_start(kKernTrainOther, stream);
                hipLaunchKernelGGL(train_move_kernel, dim3((unsigned)most(max_rows, kMoveShift), nt), dim3(kHistThreads), 0,
                                   stream, d, level - 1, turn, prm);
                prof_stop(stream);
            }
            prof_start(kKernTrainHist, stream);
            if (level == 0 || !grown) {
                // (below the root the children with fewer rows)
                const unsigned layers = (unsigned)((most(level ? max_rows / 2 : max_rows, shift) + 7) / 8);
                const unsigned emit = level == 0 && round > 0 ? 1u : 0u;
                hipLaunchKernelGGL(train_hist_kernel, dim3(8 * groups, nt, layers + emit), dim3(kHistThreads), 0, stream, d,
                                   level, turn, shift, hb, (int)layers, prm.max_depth);
            } else {
                const unsigned movers = (unsigned)most(max_rows, kMoveShift);
                const unsigned layers = (movers + 8 * groups - 1) / (8 * groups);
                hipLaunchKernelGGL(train_grow_kernel, dim3(8 * groups, nt, layers + (unsigned)((most(max_rows, shift) + 7) / 8)),
                                   dim3(kHistThreads), 0, stream, d, level - 1, turn, shift, hb, (int)layers, (int)movers, prm);
            }
            prof_stop(stream);
            prof_start(kKernTrainSplit, stream);
            const unsigned waves = parents * nt <= kSplitWideNodes ? kSplitWaves : 2;
            hipLaunchKernelGGL(train_split_kernel, dim3((unsigned)pt.max_feat, (unsigned)parents, nt),
                               dim3(64 * waves), 2 * waves * kBins * 8,
                               stream, d, level, turn, shift, hb, grown ? 1 : 0, prm);
            prof_stop(stream);
        }
        const int last = std::max(0, prm.max_depth - 1);
        const int64_t finishers = std::min<int64_t>(max_rows, (max_rows >> kMoveShift) + ((int64_t)1 << last));
        prof_start(kKernTrainOther, stream);
        hipLaunchKernelGGL(train_finish_kernel, dim3((unsigned)finishers, nt), dim3(kHistThreads), 0, stream, d, last,
                           turn, prm);
        if (round + 1 == n_rounds || prm.max_depth == 0)         // else with the next round's histograms
            hipLaunchKernelGGL(train_emit_kernel, dim3(nt), dim3(kHistThreads), 0, stream, d, prm.max_depth, turn ^ 1);
        prof_stop(stream);
        const int rc = check_launch("training kernels launch");
        if (rc != FS_OK)
            return rc;
    }
    return FS_OK;
}

}  // namespace

extern "C" int fs_train_boost(int32_t n_trainers, fs_trainer *const *trainers, int32_t n_rounds,
                              const fs_train_params *p, void *stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    int rc = check_batch("fs_train_boost", n_trainers, trainers);
    if (rc != FS_OK)
        return rc;
    if (!p)
        return fail(FS_EINVAL, "fs_train_boost: params is NULL");
    if (n_rounds < 0)
        return fail(FS_EINVAL, "fs_train_boost: n_rounds %d is negative", n_rounds);
    if (p->max_depth < 0 || p->max_depth > FS_TRAIN_MAX_DEPTH)
        return fail(FS_EUNSUPPORTED, "fs_train_boost: max_depth=%d outside 0..%d", p->max_depth,
                    FS_TRAIN_MAX_DEPTH);
    if (!(p->eta > 0.0f) || !(p->lambda >= 0.0f) || !(p->grad_scale > 0.0f) || isinf(p->grad_scale) ||
        isnan(p->min_gain) || isnan(p->min_child_weight))
        return fail(FS_EINVAL, "fs_train_boost: eta > 0, lambda >= 0, grad_scale > 0 required");
    int exp2 = 0;
    if (frexpf(p->grad_scale, &exp2) != 0.5f)
        return fail(FS_EINVAL, "fs_train_boost: grad_scale must be a power of two");
    if (n_trainers == 0 || n_rounds == 0)
        return FS_OK;
    for (int i = 0; i < n_trainers; ++i) {
        const fs_trainer *t = trainers[i];
        if (p->max_depth > t->max_depth)
            return fail(FS_EUNSUPPORTED, "fs_train_boost: trainer %d was created for max_depth %d", i, t->max_depth);
        if (t->trees_enqueued + n_rounds > t->max_trees)
            return fail(FS_EUNSUPPORTED, "fs_train_boost: trainer %d holds %d trees of at most %d", i,
                        t->trees_enqueued, t->max_trees);
    }
    Params prm;
    prm.eta = (double)p->eta;
    prm.lambda = (double)p->lambda;
    prm.min_gain = (double)p->min_gain;
    prm.inv_scale = 1.0 / (double)p->grad_scale;
    double mcw = ceil((double)p->min_child_weight);
    prm.mcw = mcw < 1.0 ? 1 : (mcw > 9e18 ? (long long)9e18 : (long long)mcw);
    prm.grad_scale = p->grad_scale;
    prm.max_depth = p->max_depth;
    try {
        // Largest families first in every launch: the last workgroups to be dispatched should be the short
        // ones.  (The order of the descriptors is internal; kernels index by block.)
        std::vector<fs_trainer *> order(trainers, trainers + n_trainers);
        std::vector<Part> parts, todo(1, make_part(order.data(), 0, n_trainers, p->max_depth));
        size_t need = 0;
        while (!todo.empty()) {                                  // halves of what is too much at a time
            const Part pt = todo.back();
            todo.pop_back();
            if (pt.n > 1 && pt.bytes > most_work()) {
                todo.push_back(make_part(order.data(), pt.first + pt.n / 2, pt.n - pt.n / 2, p->max_depth));
                todo.push_back(make_part(order.data(), pt.first, pt.n / 2, p->max_depth));
                continue;
            }
            need = std::max(need, pt.bytes);
            parts.push_back(pt);
            std::stable_sort(order.begin() + pt.first, order.begin() + pt.first + pt.n,
                             [](const fs_trainer *x, const fs_trainer *y) { return x->h.n_rows > y->h.n_rows; });
        }

        int dev = 0;
        FS_HIP(hipGetDevice(&dev));
        if (dev < 0 || dev >= 16)
            return fail(FS_EUNSUPPORTED, "device ordinal %d not supported", dev);
        // Everything that can fail for want of memory comes before the first launch: either all trainers
        // get their rounds or none.
        std::lock_guard<std::mutex> lock(g_train_mu);
        BatchBuf &b = g_batch[dev];
        if (b.work_bytes < need) {                               // an override asks for more than was reserved
            rc = grow_work(b, need, need);
            if (rc != FS_OK)
                return rc;
        }
        for (const Part &pt : parts) {
            char *at = (char *)b.work;
            for (int i = pt.first; i < pt.first + pt.n; ++i) {
                TrainDesc &h = order[(size_t)i]->h;
                size_t hist, part;
                const size_t bytes = hist_bytes(order[(size_t)i], p->max_depth, pt.shift, pt.hb, &hist, &part);
                const int planes = hist_planes(order[(size_t)i], pt.hb);
                h.hist = (unsigned long long *)at;
                h.hist_plane = (int64_t)hist;
                h.part = h.hist + planes * hist;
                h.part_plane = (int64_t)part;
                at += bytes;
            }
        }
        const TrainDesc *d = nullptr;
        rc = begin_work(b, stream);
        if (rc == FS_OK)
            rc = upload_batch(n_trainers, order.data(), stream, &d);
        for (size_t i = 0; i < parts.size() && rc == FS_OK; ++i) {
            rc = train_part(d + parts[i].first, parts[i], n_rounds, prm, stream);
            for (int k = 0; k < parts[i].n && rc == FS_OK; ++k)
                order[(size_t)(parts[i].first + k)]->trees_enqueued += n_rounds;
        }
        end_work(b, order.data(), n_trainers, stream);
        return rc;
    } catch (const std::bad_alloc &) {
        return fail(FS_ENOMEM, "out of host memory");
    }
}

extern "C" int fs_trainer_size(const fs_trainer *t, int32_t *n_trees, int64_t *n_nodes, void *stream_)
{
    if (!t)
        return fail(FS_EINVAL, "fs_trainer_size: trainer is NULL");
    FS_HIP(hipStreamSynchronize((hipStream_t)stream_));
    int32_t c[4];
    FS_HIP(hipMemcpy(c, t->h.counters, sizeof(c), hipMemcpyDeviceToHost));
    if (n_trees)
        *n_trees = c[1];
    if (n_nodes)
        *n_nodes = c[2];
    return FS_OK;
}

extern "C" int fs_trainer_export(const fs_trainer *t, int32_t *tree_off, int32_t *split_feature,
                                 float *threshold, int32_t *left, int32_t *right, float *value,
                                 void *stream_)
{
    if (!t || !tree_off || !split_feature || !threshold || !left || !right || !value)
        return fail(FS_EINVAL, "fs_trainer_export: NULL argument");
    FS_HIP(hipStreamSynchronize((hipStream_t)stream_));
    int dev = -1;
    if (hipGetDevice(&dev) == hipSuccess && dev == t->device) {  // at once, if it is small (six plain copies took 95 us)
        const Staging staging(dev, 0);
        const int32_t *at = (const int32_t *)staging.p;
        if (at) {
            hipLaunchKernelGGL(train_export_kernel, dim3(32), dim3(256), 0, nullptr, t->h, (int32_t *)staging.p,
                               (int64_t)(kStagingBytes / sizeof(int32_t)));
            const int rc = check_launch("train_export_kernel launch");
            FS_HIP(hipStreamSynchronize(nullptr));
            if (rc != FS_OK)
                return rc;
            if (at[2] != 0) {
                const size_t offs = (size_t)at[0] + 1, n = (size_t)at[1];
                at += 4;
                memcpy(tree_off, at, sizeof(int32_t) * offs);
                at += offs;
                for (void *out : {(void *)split_feature, (void *)threshold, (void *)left, (void *)right, (void *)value}) {
                    memcpy(out, at, sizeof(int32_t) * n);
                    at += n;
                }
                return FS_OK;
            }
        }
    }
    int32_t c[4];
    FS_HIP(hipMemcpy(c, t->h.counters, sizeof(c), hipMemcpyDeviceToHost));
    const size_t n = (size_t)c[2];
    FS_HIP(hipMemcpy(tree_off, t->h.m_tree_off, sizeof(int32_t) * ((size_t)c[1] + 1), hipMemcpyDeviceToHost));
    if (n) {
        FS_HIP(hipMemcpy(split_feature, t->h.m_feat, sizeof(int32_t) * n, hipMemcpyDeviceToHost));
        FS_HIP(hipMemcpy(threshold, t->h.m_thr, sizeof(float) * n, hipMemcpyDeviceToHost));
        FS_HIP(hipMemcpy(left, t->h.m_left, sizeof(int32_t) * n, hipMemcpyDeviceToHost));
        FS_HIP(hipMemcpy(right, t->h.m_right, sizeof(int32_t) * n, hipMemcpyDeviceToHost));
        FS_HIP(hipMemcpy(value, t->h.m_val, sizeof(float) * n, hipMemcpyDeviceToHost));
    }
    return FS_OK;
}

static int read_predictions(const fs_trainer *t, float *row_pred, float *prog_pred, hipStream_t stream)
{
    if (prog_pred) {
        const TrainDesc *d = nullptr;
        int rc = upload_batch(1, &t, stream, &d);
        if (rc != FS_OK)
            return rc;
        launch_grad(d, t->h.n_programs, 1, 1.0f, 0, 0, stream);
        rc = check_launch("train_grad_kernel launch");
        if (rc != FS_OK)
            return rc;
        FS_HIP(hipMemcpyAsync(prog_pred, t->h.prog_pred, sizeof(float) * (size_t)t->h.n_programs,
                              hipMemcpyDeviceToDevice, stream));
    }
    if (row_pred)
        FS_HIP(hipMemcpyAsync(row_pred, t->h.row_pred, sizeof(float) * (size_t)t->h.n_rows,
                              hipMemcpyDeviceToDevice, stream));
    return FS_OK;
}

extern "C" int fs_trainer_predictions(const fs_trainer *t, float *row_pred, float *prog_pred, void *stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (!t)
        return fail(FS_EINVAL, "fs_trainer_predictions: trainer is NULL");
    fs_trainer *tt = const_cast<fs_trainer *>(t);
    int rc = check_batch("fs_trainer_predictions", 1, &tt);
    if (rc != FS_OK)
        return rc;
    std::lock_guard<std::mutex> lock(g_train_mu);
    if (t->device < 0 || t->device >= 16)                        // (its memory is never kept)
        return read_predictions(t, row_pred, prog_pred, stream);
    BatchBuf &b = g_batch[t->device];
    rc = begin_work(b, stream);
    if (rc == FS_OK)
        rc = read_predictions(t, row_pred, prog_pred, stream);
    end_work(b, &tt, 1, stream);
    return rc;
}
