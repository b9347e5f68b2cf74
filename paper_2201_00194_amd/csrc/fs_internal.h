// Internal declarations shared by the library's translation units (not installed).
#ifndef FS_INTERNAL_H
#define FS_INTERNAL_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "familyseer.h"
#include "fs_treelet.h"

namespace fs {

// ---- error reporting ---------------------------------------------------------------------
int fail(int code, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
int fail_hip(hipError_t e, const char *what);

#define FS_HIP(call)                                   \
    do {                                               \
        hipError_t fs_e_ = (call);                     \
        if (fs_e_ != hipSuccess)                       \
            return ::fs::fail_hip(fs_e_, #call);       \
    } while (0)

// ---- test and tuning overrides (fs_tune_set); -1 = automatic ---------------------------------
int tune(int option);

// ---- device-side model formats -------------------------------------------------------------

// Node of the reference device layout (global memory).  One entry per node, trees
// concatenated in the caller's numbering, child ids already offset to global node indices.
//   x: bits of threshold (internal) or of the leaf value (leaf)
//   y: split feature, or -1 at a leaf
//   z: global index of the left child    w: of the right child
typedef int4 GNode;

// ---- LDS-staged model format -------------------------------------------------------------------
// The ensemble is cut into chunks of consecutive trees.  A chunk is a byte image that is copied
// verbatim to LDS offset 0:
//     [run records of the wavefront slots] [further run records] [nodes ...]   (multiple of 16)
// A node is 8 bytes {w0, w1}:
//     internal: w0 = threshold bits, w1 = (feature * 256) << 16 | byte offset of the LEFT child;
//               the right child sits right after the left one
//     leaf:     w0 = value bits,     w1 = (n_features * 256) << 16 | (own offset - 8):
//               it reads the all-NaN column, fails '<' and so steps back onto itself
// In "compact" chunks (every tree of the model perfect and of one depth >= 1) leaves are 4-byte
// values only, laid out after the tree's internal nodes; the last split level then steps by 4.
//
// Walk order.  The wavefronts that share a tile ("slots") split the chunk's trees.  Trees are
// sorted by depth and cut into runs of at most 8 trees of similar depth; a run is walked side by
// side, to the depth of its first (deepest) tree, and the runs are dealt to the slots so that the
// slots have about the same work.  A run record is kRunWords uint32: word 0 = number of trees
// (bits 0-3) | index of the slot's next run record + 1, or 0 (bits 4-15) | depth (bits 16-31);
// words 1..8 = the run's trees: LDS offset of the root (bits 0-15) | index of the tree in its
// chunk, i.e. the place the ordered sum gives it (bits 16-23); unused tree words repeat the first.
// Record s (s < kLdsMaxWaves) is the first run of slot s (no trees: the slot is idle).
constexpr int kRunWords = 9;
constexpr int kRunBytes = 4 * kRunWords;

struct ChunkHdr {
    uint32_t byte_off;    // into the packed image
    uint32_t bytes;       // multiple of 16
    uint32_t n_trees;
    uint32_t depth;       // split levels of the deepest tree of the chunk
    uint32_t first_tree;  // model-wide index of the chunk's first tree
    uint32_t slot_off;    // into the id map: entry [slot_off + (lds byte offset >> 2)]
    uint32_t pad0;
    uint32_t pad1;
};

// LDS map of the traversal kernel (bytes):
//   [0, chunk bytes)                       model chunk (run records, nodes)
//   [tile0 - n_trees*tiles*256, tile0)     leaf values [tree in chunk][tile][lane] (fp32)
//   [tile0, 160 KB)                        `tiles` feature tiles of (n_features+1)*256 bytes,
//                                          tile0 = 160 KB - tiles * tile bytes
// Two workgroup shapes.  "small": half a compute unit's LDS, 6 wavefronts, one tile -- two
// such workgroups share a compute unit, so one walks while the other is busy with barriers,
// the ordered sum or the next chunk.  "big": the whole LDS, 12 wavefronts, 1-3 tiles -- for
// models whose trees are too large to give a small workgroup enough trees per chunk.
constexpr int kLdsModes = 2;
constexpr int kLdsModeBytes[kLdsModes] = {80 * 1024, 160 * 1024};
constexpr int kLdsModeWaves[kLdsModes] = {6, 12};
constexpr int kLdsMaxWaves = 12;
constexpr int kLdsMaxTiles = 3;         // 64-row tiles per workgroup (1, 2 or 3)
constexpr int kMaxChunkBytes = 65536 - 16;
constexpr int kMaxChunkTrees = 96;
constexpr int kPrefetchRegs = 6;        // 16-byte registers per thread for the next chunk

// Forms of the treelet traversal: two 4-tile workgroups per compute unit, or one workgroup of 12
// wavefronts that share 4, 2 or 1 tiles.
enum { kTreeletPair = 0, kTreeletSpread4 = 1, kTreeletSpread2 = 2, kTreeletSpread1 = 3, kTreeletForms = 4 };
constexpr int kTreeletFormTiles[kTreeletForms] = {4, 4, 2, 1};

}  // namespace fs

// The opaque model: host copy of what validation needs plus device arrays.
struct fs_model {
    int32_t n_features;
    int32_t n_trees;
    int64_t n_nodes;
    float bias;
    int device;
    fs::GNode *d_nodes;    // [n_nodes]
    int32_t *d_tree_off;   // [n_trees + 1]
    // LDS-staged format (absent if the model does not fit it)
    bool lds_ok;
    bool compact;          // perfect trees of one depth, 4-byte leaves
    int32_t lds_mode;      // workgroup shape chosen for this model (index into kLdsMode*)
    int32_t lds_tiles;     // 64-row tiles per workgroup chosen for this model
    int32_t lds_tile0;     // LDS byte offset of the first feature tile
    float lds_group_us;    // the planner's estimate of one tile group's time in the LDS kernel
    int32_t n_chunks;
    uint8_t *d_image;      // all chunk images back to back
    fs::ChunkHdr *d_chunks;
    uint16_t *d_slot_ids;  // caller's local node id per 4-byte slot (leaves only meaningful)
    size_t image_bytes;
    // Rank-coded format (deep perfect trees): features become 16-bit ranks among the model's
    // own thresholds of that feature, nodes shrink to 4 bytes (see fs_rank.hip)
    bool rank_ok;
    int32_t rk_depth;          // common depth of the trees
    int32_t rk_tree_bytes;     // of a tree in LDS: heap words 1 .. 2^(depth - 1) - 1, word 0 unused, whole 16 bytes
    int32_t rk_forced_tiles;   // tiles per workgroup as overridden, or 0
    uint32_t *d_rk_nodes;      // [n_trees][rk_tree_bytes], then [n_trees][2^(depth - 1)] RankLast
    uint16_t *d_rk_ids;        // [n_trees][2^(depth+1)] 1-based heap order: caller's local node id
    float *d_cuts;             // [n_features][2^cut_bits]: the feature's sorted distinct
                               // thresholds, NaN-padded, as a breadth-first search tree; or, with
                               // cut_bits negative, [n_features][-cut_bits bytes]: RankColumn tables
    int32_t cut_bits;
    int32_t bin_group;         // features whose tables a workgroup of the coder holds
    // Byte-rank treelets (fs_treelet.h); null if the model does not fit that format
    bool tl_ok;
    bool tl_pair;              // two chunk buffers fit half a compute unit's LDS
    int32_t tl_cols;
    // a round of workgroups, estimated, us (spread forms: the whole call); [row-major input][form].  A model
    // with tl_ok and lds_ok has both walks, and the call chooses (fs_forms.h)
    float tl_us[2][fs::kTreeletForms];
    float tl_once_us;          // and once per call of the pair form
    void *d_tl_data;           // everything of this format, one allocation
    fs::TreeletModel *d_tl;    // inside it
};

namespace fs {

struct RankShape {                       // a workgroup of the rank walk
    int32_t tiles;                       // of 64 rows
    int32_t slots, per_slot;             // wavefronts of a tile that have trees, and how many at a time
    int32_t tile0;                       // LDS byte offset of the first (u16) tile
};

// ---- per-family descriptor as the kernels see it --------------------------------------------
struct FamDesc {
    const GNode *nodes;
    const int32_t *tree_off;
    const float *features;
    const int32_t *prog_off;
    float *prog_score;
    float *row_score;      // never NULL on the device: caller's buffer or library scratch
    uint16_t *leaf_idx;    // may be NULL
    int32_t n_trees;
    int32_t n_features;
    int32_t layout;
    int32_t n_rows;
    int32_t n_programs;
    float bias;
    int32_t trav_block0;   // first block of the global-memory traversal grid of this family
    int32_t seg_block0;    // first block of the segmented-sum grid
    // LDS-staged traversal
    const uint8_t *image;
    const ChunkHdr *chunks;
    const uint16_t *slot_ids;
    int32_t n_chunks;
    int32_t lds_tile0;
    int32_t lds_tiles;
    int32_t compact;
    int32_t lds_block0[kLdsModes];   // first block of this family in each LDS launch
    // rank-coded traversal
    const uint32_t *rk_nodes;
    const uint16_t *rk_ids;
    const float *cuts;
    uint16_t *ranks;                 // scratch: rank-coded feature tiles [tile][feature][64]
    RankShape rk;
    int32_t rk_depth, rk_tree_bytes;
    int32_t rk_block0;               // first block of the rank traversal grid
    int32_t bin_block0;              // first block of the rank-coding grid
    int32_t bin_groups;              // feature groups of this family in the rank-coding grid
    int32_t bin_feats_per_group;
    int32_t bin_tiles_per_block;
    // row-major input: re-tiled into scratch before the LDS kernels (features then points there)
    const float *rowmajor_src;
    int32_t retile_block0;           // first block of the re-tiling grid
    int32_t retile_colblocks;        // column blocks per tile (0: family not re-tiled)
    int32_t cut_bits;                // threshold tables are padded to 2^cut_bits entries; negative: RankColumn tables of
                                     // so many bytes
    const TreeletModel *tl;          // byte-rank treelets
    int32_t tl_block0[2];            // first block of this family in the two treelet launches
};

// Descriptors reach a kernel by value, as its last argument, where a call has few of them: a call of two or three
// short kernels otherwise pays for another launch that only stores them (scoring and cutting 320 / 4096
// programs 30.6 / 35.5 us, so 27.8 / 31.9).  As many as fit do: the arguments of a kernel take 4 KB, of which 256 bytes
// are hidden ones and some are for pointers and numbers (64 cuts of 320 entries in a call, one after the other: 4.9 us,
// 7.2 from memory; 16 of them 4.8).  More descriptors lie in device memory at `far`.
constexpr size_t kNearBytes = 3600;
template <class T>
constexpr int kNear = (int)(kNearBytes / sizeof(T));
constexpr int kNearFams = kNear<FamDesc>;
struct NearFams {
    FamDesc d[kNearFams];
};
struct FamArgs1 {              // arguments of kernels with one, two and three numbers
    const FamDesc *far;
    int a;
    NearFams near;
};
struct FamArgs2 {
    const FamDesc *far;
    int a, b;
    NearFams near;
};
struct FamArgs3 {
    const FamDesc *far;
    int a, b, c;
    NearFams near;
};
static_assert(sizeof(FamArgs3) + 256 <= 4096, "kernel arguments are 4 KB at most, hidden ones among them");

// What the launchers take: descriptors in device memory or, where far is null, n of them at `host`.
template <class T>
struct Descs {
    const T *far;
    const T *host;
    int n;
};
// In a kernel: the descriptors, read-only memory either way so that they come through scalar loads; `at`: where the
// by-value ones lie among the kernel's arguments, which are laid out like a struct.
template <class T>
__device__ __forceinline__ const T *where_descs(const T *far, uint32_t at)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const uintptr_t near = (uintptr_t)__builtin_amdgcn_kernarg_segment_ptr() + at;
    return (const T *)(__attribute__((address_space(4))) const T *)(far ? (uintptr_t)far : near);
#else
    (void)at;
    return far;
#endif
}
template <class Near, class T>
Near near_descs(const Descs<T> &from)
{
    Near near;
    if (!from.far)
        for (int i = 0; i < from.n; ++i)
            near.d[i] = from.host[i];
    return near;
}

// One workgroup of the first top-k stage: the whole request, or one slice of a large one.
struct TopkDesc {
    const float *score;
    int32_t *out_idx;
    float *out_score;      // may be NULL
    int32_t n;             // entries of the request
    int32_t k;
    int32_t sub_begin, sub_end;      // the slice [sub_begin, sub_end) this workgroup ranks
    unsigned long long *comp_out;    // NULL: final answer to out_idx/out_score; else the slice's
                                     // best min(k, slice length) (key, ~index) composites, best first
    int32_t comp_pad;                // 1: pad comp_out with 0 up to k entries
    int32_t pad;
};

// Second stage of a large request: merge the slices' candidates.
struct TopkMergeDesc {
    const unsigned long long *comp_in;   // n_comp composites (0 = padding)
    const float *score;
    int32_t *out_idx;
    float *out_score;      // may be NULL
    int32_t n_comp;
    int32_t n;             // entries of the request
    int32_t k;
    int32_t pad;
};


// One merge of up to kTopkWays lists of composites (each best first) in global memory: the best `lo` of
// their union go to `out` (composites), or, at the last level of a request, to its
// out_idx / out_score (then `lo` = min(n, k) and entries up to k are padded with -1 / -inf).
constexpr int kTopkWays = 8;
struct TopkJoinDesc {
    const unsigned long long *list[kTopkWays];   // readable also where `len` is 0
    unsigned long long *out;       // NULL at the last level
    const float *score;
    int32_t *out_idx;
    float *out_score;              // may be NULL
    int32_t len[kTopkWays];
    int32_t n, longest, lo, k;     // lists, entries of the longest
};

// u16 rank tiles keep the features of a row in pairs: features 2i and 2i+1 of row l share the
// 32-bit word at i*256 + 4*l of the tile, so that lane l always reads from LDS bank l whichever
// feature it asks for (with one u16 column after the other, two lanes would meet in every bank).
// A tile therefore has an even number of columns.
__host__ __device__ inline int rank_tile_cols(int n_features) { return (n_features + 1) & ~1; }
__host__ __device__ inline uint32_t rank_feature_offset(int f) { return (uint32_t)(f >> 1) * 256u + (uint32_t)(f & 1) * 2u; }

// (64 workgroups, 75 merges, 25 joins)
constexpr int kNearTopk = kNear<TopkDesc>, kNearMerge = kNear<TopkMergeDesc>, kNearJoins = kNear<TopkJoinDesc>;
struct NearTopk {
    TopkDesc d[kNearTopk];
};
struct NearMerge {
    TopkMergeDesc d[kNearMerge];
};
struct NearJoins {
    TopkJoinDesc d[kNearJoins];
};

// ---- launchers (each returns FS_OK or records an error) ---------------------------------------
int launch_traverse_global(const FamDesc *d_desc, int n_families, int total_blocks,
                           hipStream_t stream);
int launch_traverse_lds(const Descs<FamDesc> &descs, int mode, int total_blocks,
                        int groups_per_wg, bool dump, hipStream_t stream);
// Tile groups one workgroup of the LDS traversal takes in a row; host (workgroup counts) and
// kernel agree on it through this function.  From its second group on a workgroup receives the
// tiles through registers, kLdsTileRegs 16-byte pieces per thread, so `want` only holds for
// column-blocked input whose `tiles` tiles fit there; other families get one group per workgroup.
constexpr int kLdsTileRegs = 7;
__host__ __device__ inline int lds_groups_per_wg(int layout, int n_features, int tiles, int threads,
                                                 int want)
{
    if (layout != FS_COLBLOCK64 || tiles * n_features * 16 > kLdsTileRegs * threads)
        return 1;
    return want < 1 ? 1 : want;
}
int launch_rank_code(const FamDesc *d_desc, int n_families, int total_blocks, hipStream_t stream);
// `regs`: most 16-byte pieces of a slot's trees that a thread copies.
int launch_traverse_rank(const FamDesc *d_desc, int n_families, int total_blocks, int regs, bool dump,
                         hipStream_t stream);
// `launch`: which of FamDesc::tl_block0 numbers the blocks (a call makes up to two launches: models whose
// chunks only fit a whole compute unit's LDS cannot take the first form).
int launch_treelet(const Descs<FamDesc> &descs, int launch, int form, int total_blocks, bool dump,
                   hipStream_t stream);
// rows, programs: of all families
int launch_segsum(const Descs<FamDesc> &descs, int64_t rows, int64_t programs, int total_blocks, hipStream_t stream);
// max_entries: of a workgroup
int launch_topk(const Descs<TopkDesc> &descs, int max_k, int max_entries, hipStream_t stream);
// max_padded: largest (slices * k rounded up to a power of two) over the requests
int launch_topk_merge(const Descs<TopkMergeDesc> &descs, int max_padded, hipStream_t stream);
constexpr int kTopkSliceMin = 8192;      // requests at least this long are split into slices,
constexpr int kTopkAtOnce = 16384;       // but not up to this long with a small cut, in calls without longer ones: a workgroup
constexpr int kTopkSmallCut = 256;       // holds so many keys, and there is no second kernel then.  Five cuts of 50 of 9001 12.1
                                         // us in slices and 9.6 so, eight of 128 of 10 000 13.5 and 11.0, of 256 14.5 and
                                         // 11.5, four of 256 of 16 384 17.5 and 12.4; beside one of 65 536 14.5 and 16.8
constexpr int kTopkSliceEntries = 2048;  // of at least this many entries
constexpr int kTopkMaxSlices = 16;
constexpr int kTopkMergeCap = 16384;     // composites (lists padded to a power of two) the merge holds in LDS
constexpr int kTopkWideSlice = 2048;     // slice length of cuts too wide for the LDS merge (k > 4096)
constexpr int kTopkWideMaxSlices = 128;
// How a top-k request of n entries and cut k is served:
//   mode 0  one workgroup, finished by the first kernel;
//   mode 1  long request, k <= 4096: `s` slices of `per` entries (one workgroup each) leave their
//           best k in scratch and one workgroup merges them in LDS;
//   mode 2  long request with a wider cut: slices of about kTopkWideSlice entries leave their best
//           min(k, length) sorted, then merges of kTopkWays lists in global memory, level by level.
struct TopkPlan { int mode, s, per; };
// `whole`: no request of the call needs slices whatever the others do (topk_whole).
inline bool topk_whole(int n, int k) { return n < kTopkSliceMin || k == 0 || (n <= kTopkAtOnce && k <= kTopkSmallCut); }
inline TopkPlan topk_plan(int n, int k, bool whole)
{
    TopkPlan p = {0, 1, n};
    if (whole || n < kTopkSliceMin || k == 0)
        return p;
    int kp = 1;
    while (kp < k)
        kp <<= 1;
    if (kp > kTopkMergeCap / 4) {
        int s = (n + kTopkWideSlice - 1) / kTopkWideSlice;
        if (s > kTopkWideMaxSlices)
            s = kTopkWideMaxSlices;
        if (s >= 2) {
            p.mode = 2;
            p.s = s;
            p.per = (((n + s - 1) / s) + 63) & ~63;
        }
        return p;
    }
    int s = kTopkMergeCap / kp;
    if (s > kTopkMaxSlices)
        s = kTopkMaxSlices;
    if (s > n / kTopkSliceEntries)
        s = n / kTopkSliceEntries;
    if (s >= 2) {
        p.mode = 1;
        p.s = s;
        p.per = (((n + s - 1) / s) + 63) & ~63;
    }
    return p;
}
int launch_topk_joins(const Descs<TopkJoinDesc> &descs, int max_entries, hipStream_t stream);
int launch_retile(const FamDesc *d_desc, int n_families, int total_blocks, hipStream_t stream);
int launch_pack_colblock64(const float *in, int64_t n_rows, int32_t n_features, float *out,
                           hipStream_t stream);

// Frees what training keeps on a device without trainers, for a caller that ran out of device memory; true
// if there was something (fs_train.hip).
bool give_back_training_memory(int device);
// hipMalloc on the current device that does so before it gives up.
hipError_t device_malloc(void **p, size_t bytes);

// ---- optional per-kernel timing (fs_profile_begin / fs_profile_end) ----------------------------
enum KernelClass { kKernTraverse = 0, kKernSegsum = 1, kKernTopk = 2, kKernPack = 3,
                   kKernTraverseGlobal = 4, kKernRankCode = 5, kKernTraverseRank = 6,
                   kKernTrainHist = 7, kKernTrainSplit = 8, kKernTrainOther = 9,
                   kKernClasses = 10 };
// Records an event pair around the launches made between prof_start and prof_stop when
// profiling is on; no-ops otherwise.  Both run under the API mutex.
void prof_start(int kernel_class, hipStream_t stream);
void prof_stop(hipStream_t stream);

// rank-coding kernel: most tiles handled by one workgroup, LDS bytes for threshold tables
constexpr int kBinTilesPerBlock = 256;
constexpr int kBinTableBytes = 80 * 1024;    // two workgroups fit a compute unit
constexpr int kBinTreeBytes = 64 * 1024;     // of search trees
// Head of a feature's table, if values are coded by buckets: then 16-bit numbers of the thresholds in lower buckets
// for each bucket, then the sorted thresholds, NaN behind.  The bucket of x is x * scale + offset (one rounding),
// truncated and clamped, which never decreases with x; up to 2^steps - 1 thresholds share one.
struct RankColumn {
    float scale, offset;
    int32_t buckets, steps;
};
constexpr int kRankMostSteps = 4;
constexpr int kRankWaves = 16;
constexpr int kRankLdsBytes = 160 * 1024;
constexpr int kRankMostTrees = 8;        // of a slot
constexpr int kRankSay = 16;             // families of at least a 16th of the longest's tiles decide about the kernel's registers
struct RankLast {                        // a split of a tree's last level, as in LDS, and its leaves' values
    uint32_t split;
    float left, right;
};
// For a family of own_tiles in a launch of all_tiles; no tiles where a tree does not fit beside one.
RankShape rank_shape(int n_features, int n_trees, int tree_bytes, int64_t own_tiles, int64_t all_tiles, int forced_tiles);

// Tiles of up to 2^31 - 1 rows.
__host__ __device__ inline int row_tiles(int n_rows) { return (int)(((uint32_t)n_rows + 63u) >> 6); }

constexpr int kTravRowsPerBlock = 256;   // rows per block of the global-memory traversal
constexpr int kSegProgsPerBlock = 256;   // programs per block of the segmented sum

}  // namespace fs
#endif
