// Rank-coded scoring for models of deep perfect trees.
//
// A split "x[f] < thr" only asks how x[f] orders against the thresholds the model itself
// uses on feature f.  Let cuts_f be those thresholds, sorted and distinct, and
//     rank(x) = number of cuts_f that are <= x            (NaN: 65535)
//     rank(thr) = 1 + position of thr in cuts_f           (NaN threshold: 0)
// then  x < thr  <=>  rank(x) < rank(thr), exactly: the walk over 16-bit ranks reaches the
// same leaves as the walk over the fp32 values (Section 4.2 of the paper: the family's model
// estimates each candidate; nothing in the estimate changes).  What it buys: a feature tile
// takes 2 bytes per value instead of 4 and a split node 4 bytes instead of 8, so a compute
// unit's LDS holds twice the rows and twice the trees -- deep trees otherwise leave room for
// only a handful of trees per chunk and the model has to stream through LDS once per 128 rows.
//
// Two kernels:
//   rank_code_kernel     fp32 feature tiles -> u16 rank tiles (searches in LDS-resident
//                        threshold tables, one feature group per workgroup)
//   traverse_rank_kernel the LDS-staged walk over rank tiles; trees in heap order without
//                        child pointers (node i has children 2i, 2i+1, 1-based), the last level of
//                        splits and the leaves in memory; the wavefronts that share a tile walk
//                        trees of their own and pass the row's sum on in tree order
#include <algorithm>

#include "fs_internal.h"
#include "fs_lds.h"

namespace fs {

// ------------------------------------------------------------------------------------------------
// rank coding
// ------------------------------------------------------------------------------------------------
constexpr int kBinThreads = 1024;

// Every feature's thresholds are padded with NaN to 2^q - 1 keys (q the same for all features
// of a model) and stored as an implicit search tree in breadth-first order (word 0 unused,
// node i has children 2i and 2i+1).  The count of keys <= x is then a branch-free descent
// with q fixed steps,   i = 2i + (key[i] <= x),   rank = i - 2^q   (NaN padding never compares
// <=).  Breadth-first order matters on this memory: the nodes of one level are neighbours, so
// the lanes' reads spread over the LDS banks, whereas the probes of a bisection of the sorted
// array are a power-of-two stride apart and all fall into the same bank.  Four searches run
// interleaved per wavefront.
//
// Where the thresholds are spread well enough (bucket_tables), the tree's upper levels give way to a bucket table: a
// multiply-add finds the bucket, the table the thresholds below it, and a bisection of at most 4 steps the bucket's own.
// (With q = 12 steps of four instructions vector issue took 95 % of the clocks.  2.1 M rows of 164 features, 3100 thresholds
// each, 2.1 GB: 611 us, by buckets 490, see below for what is left of that.)
constexpr int kBinChains = 4;

template <int N> struct RankInt { static constexpr int value = N; };

// Column-blocked rows by buckets: a wavefront takes four features at a time over all its tiles, so that what the
// features' tables say is read once and the loop is vector and LDS instructions.  (Feature by feature within a tile the
// loop had 40 scalar instructions a search beside 26 vector ones, and scalar loads among its LDS reads:
// 2.1 M rows of 164 features, 3100 thresholds each, 488 us, so 392; the bytes take 322.)
template <int STEPS>
__device__ __forceinline__ void code_by_buckets(const FamDesc &d, int f0, int gf, int len, int t0, int nt, int wave, int lane)
{
    constexpr int kWaves = kBinThreads / 64;
    const int F = d.n_features;
    const uint32_t tile_words = (uint32_t)rank_tile_cols(F) * 32u;            // of a tile of ranks
    for (int j0 = 0; j0 < gf; j0 += kBinChains) {
        float scale[kBinChains], offset[kBinChains];
        uint32_t lut[kBinChains], keys[kBinChains], most = 0;
        uint32_t from[kBinChains];
#pragma unroll
        for (int k = 0; k < kBinChains; ++k) {
            const int j = min(j0 + k, gf - 1);
            auto col = FS_CONST(RankColumn, d.cuts + (int64_t)(f0 + j) * len);
            scale[k] = col->scale;
            offset[k] = col->offset;
            most = (uint32_t)col->buckets - 1u;                              // the same for all features
            lut[k] = 4u * (uint32_t)(j * len) + 16u;
            keys[k] = lut[k] + 2u * (most + 1u);
            from[k] = 64u * (uint32_t)(f0 + j);
        }
        const int n = min(kBinChains, gf - j0);
        auto X = FS_GLOBAL(const float, d.features) + (int64_t)t0 * F * 64 + lane;
        auto R = FS_GLOBAL(uint16_t, d.ranks) + (int64_t)t0 * tile_words * 2 + 2 * lane;
        float next[kBinChains] = {};
        if (wave < nt)
#pragma unroll
            for (int k = 0; k < kBinChains; ++k)
                next[k] = X[(int64_t)wave * F * 64 + from[k]];
        for (int t = wave; t < nt; t += kWaves) {
            float x[kBinChains];
            uint32_t at[kBinChains], r[kBinChains];
#pragma unroll
            for (int k = 0; k < kBinChains; ++k)
                x[k] = next[k];
            const int64_t ahead = (int64_t)min(t + kWaves, nt - 1) * F * 64;
#pragma unroll
            for (int k = 0; k < kBinChains; ++k)
                next[k] = X[ahead + from[k]];
#pragma unroll
            for (int k = 0; k < kBinChains; ++k)
                at[k] = lds_u16(lut[k] + 2u * min(to_u32(__builtin_fmaf(x[k], scale[k], offset[k])), most));
#pragma unroll
            for (int k = 0; k < kBinChains; ++k)
                at[k] = keys[k] + 4u * at[k];                                // the first threshold that is not known to be <= x
#pragma unroll
            for (int s = STEPS - 1; s >= 0; --s) {
                float c[kBinChains];
#pragma unroll
                for (int k = 0; k < kBinChains; ++k)
                    c[k] = lds_f(at[k] + (4u << s) - 4u);
#pragma unroll
                for (int k = 0; k < kBinChains; ++k)
                    at[k] += c[k] <= x[k] ? 4u << s : 0u;
            }
#pragma unroll
            for (int k = 0; k < kBinChains; ++k)
                r[k] = x[k] != x[k] ? 65535u : (at[k] - keys[k]) >> 2;
            const int64_t base = (int64_t)t * tile_words * 2;                 // u16 units
            if (n == kBinChains) {                           // features 2i and 2i + 1 share a word of the tile (f0 is a multiple of 4)
#pragma unroll
                for (int k = 0; k < kBinChains; k += 2)
                    *(__attribute__((address_space(1))) uint32_t *)(R + base + (rank_feature_offset(f0 + j0 + k) >> 1)) = r[k] | r[k + 1] << 16;
            } else {
#pragma unroll
                for (int k = 0; k < kBinChains; ++k)
                    if (k < n)
                        R[base + (rank_feature_offset(f0 + j0 + k) >> 1)] = (uint16_t)r[k];
            }
        }
    }
}

__global__ void __launch_bounds__(kBinThreads, 8)     // two workgroups per compute unit
rank_code_kernel(const FamDesc *__restrict__ descs, int n_families)
{
    int lo = 0, hi = n_families - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (descs[mid].bin_block0 <= (int)blockIdx.x)
            lo = mid;
        else
            hi = mid - 1;
    }
    const FamDesc &d = descs[lo];
    const int local = blockIdx.x - d.bin_block0;
    const int group = local % d.bin_groups, tile_block = local / d.bin_groups;
    const int F = d.n_features;
    const int f0 = group * d.bin_feats_per_group;
    const int gf = min(d.bin_feats_per_group, F - f0);
    const int n_tiles = row_tiles(d.n_rows);
    const int tpb = d.bin_tiles_per_block;
    const int t0 = tile_block * tpb;
    const int nt = min(tpb, n_tiles - t0);
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int q = d.cut_bits;                       // table stride 2^q entries
    const bool bucketed = q < 0;
    const int len = bucketed ? -q / 4 : 1 << q;     // words of a feature's table

    // this group's padded threshold tables: one contiguous, 16-byte aligned run, straight from
    // memory to LDS (what is left below 64 pieces goes through a register)
    {
        auto cuts = FS_GLOBAL(const u32x4, d.cuts + (int64_t)f0 * len);
        const int n16 = gf * len / 4;
        const int rest = lds_fill_direct(cuts, 0u, n16, wave, kBinThreads / 64, lane) + tid;
        if (rest < n16)
            lds_store_u4(16u * (uint32_t)rest, cuts[rest]);
        lds_direct_wait();
    }
    __syncthreads();

    if (bucketed && d.layout != FS_ROWMAJOR) {
        switch (FS_CONST(RankColumn, d.cuts)->steps) {               // the same for all features
        case 0: code_by_buckets<0>(d, f0, gf, len, t0, nt, wave, lane); break;
        case 1: code_by_buckets<1>(d, f0, gf, len, t0, nt, wave, lane); break;
        case 2: code_by_buckets<2>(d, f0, gf, len, t0, nt, wave, lane); break;
        case 3: code_by_buckets<3>(d, f0, gf, len, t0, nt, wave, lane); break;
        default: code_by_buckets<kRankMostSteps>(d, f0, gf, len, t0, nt, wave, lane);
        }
        return;
    }

    auto X = FS_GLOBAL(const float, d.features);
    auto R = FS_GLOBAL(uint16_t, d.ranks);
    // A wavefront takes tiles wave, wave+16, ... of the block and, per tile, the group's
    // features four at a time (one search chain each).  The next round's values are fetched
    // while the current round is searched.
    const int n_waves = kBinThreads / 64;
    const int rounds_per_tile = (gf + kBinChains - 1) / kBinChains;
    // Element (tile, feature f0 + j, lane) of the input: column-blocked tiles, or row-major rows
    // (the row index is clamped: the last tile of a row-major matrix has no padding rows).
    const bool rowmajor = d.layout == FS_ROWMAJOR;
    auto x_at = [&](int tile, int j) -> int64_t {
        if (rowmajor)
            return (int64_t)min(tile * 64 + lane, d.n_rows - 1) * F + f0 + j;
        return ((int64_t)tile * F + f0 + j) * 64 + lane;
    };
    int t = wave, jg = 0;                            // current round: tile t, features 4*jg..
    float xn[kBinChains];
    if (t < nt) {
#pragma unroll
        for (int k = 0; k < kBinChains; ++k)
            xn[k] = X[x_at(t0 + t, min(k, gf - 1))];
    }
    while (t < nt) {
        const int j0 = jg * kBinChains;
        const int64_t base = (int64_t)(t0 + t) * rank_tile_cols(F) * 64 + 2 * lane;   // u16 units
        float x[kBinChains];
        uint32_t r[kBinChains], tab[kBinChains];
#pragma unroll
        for (int k = 0; k < kBinChains; ++k) {
            x[k] = xn[k];
            tab[k] = 4u * (uint32_t)(min(j0 + k, gf - 1) * len);
        }
        // next round
        int tn = t, jn = jg + 1;
        if (jn == rounds_per_tile) {
            jn = 0;
            tn = t + n_waves;
        }
        if (tn < nt) {
#pragma unroll
            for (int k = 0; k < kBinChains; ++k)
                xn[k] = X[x_at(t0 + tn, min(jn * kBinChains + k, gf - 1))];
        }
        if (bucketed) {
            int steps = 0;
            uint32_t keys[kBinChains];
#pragma unroll
            for (int k = 0; k < kBinChains; ++k) {
                auto col = FS_CONST(RankColumn, d.cuts + (int64_t)(f0 + min(j0 + k, gf - 1)) * len);
                const uint32_t bucket = to_u32(__builtin_fmaf(x[k], col->scale, col->offset));
                r[k] = lds_u16(tab[k] + 16u + 2u * min(bucket, (uint32_t)col->buckets - 1u));
                keys[k] = tab[k] + 16u + 2u * (uint32_t)col->buckets;
                steps = col->steps;                  // the same for all features
            }
            for (int s = steps - 1; s >= 0; --s) {
                float c[kBinChains];
#pragma unroll
                for (int k = 0; k < kBinChains; ++k)
                    c[k] = lds_f(keys[k] + 4u * r[k] + (4u << s) - 4u);
#pragma unroll
                for (int k = 0; k < kBinChains; ++k)
                    r[k] += c[k] <= x[k] ? 1u << s : 0u;
            }
        } else {
#pragma unroll
            for (int k = 0; k < kBinChains; ++k)
                r[k] = 1u;                           // node of the implicit search tree
            for (int s = 0; s < q; ++s) {
                float c[kBinChains];
#pragma unroll
                for (int k = 0; k < kBinChains; ++k)
                    c[k] = lds_f(tab[k] + 4u * r[k]);
#pragma unroll
                for (int k = 0; k < kBinChains; ++k)
                    r[k] = 2u * r[k] + ((c[k] <= x[k]) ? 1u : 0u);
            }
#pragma unroll
            for (int k = 0; k < kBinChains; ++k)
                r[k] -= (uint32_t)len;
        }
#pragma unroll
        for (int k = 0; k < kBinChains; ++k)
            r[k] = x[k] != x[k] ? 65535u : r[k];
        if ((f0 & 1) == 0) {
            // chains 2i and 2i+1 hold the two features of one word of the tile
            auto R2 = FS_GLOBAL(uint32_t, d.ranks);
#pragma unroll
            for (int k = 0; k < kBinChains; k += 2) {
                const int64_t at = base + (rank_feature_offset(f0 + j0 + k) >> 1);   // even
                if (j0 + k + 1 < gf)
                    R2[at >> 1] = r[k] | (r[k + 1] << 16);
                else if (j0 + k < gf)
                    R[at] = (uint16_t)r[k];
            }
        } else {
#pragma unroll
            for (int k = 0; k < kBinChains; ++k)
                if (j0 + k < gf)
                    R[base + (rank_feature_offset(f0 + j0 + k) >> 1)] = (uint16_t)r[k];
        }
        t = tn;
        jg = jn;
    }
}

int launch_rank_code(const FamDesc *d_desc, int n_families, int total_blocks, hipStream_t stream)
{
    static bool configured[16] = {};
    int dev = 0;
    FS_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 16 || !configured[dev]) {
        hipFuncAttributes attr;
        FS_HIP(hipFuncGetAttributes(&attr, (const void *)rank_code_kernel));
        if (attr.sharedSizeBytes != 0)
            return fail(FS_EDEVICE, "rank_code_kernel was built with %zu bytes of static LDS",
                        (size_t)attr.sharedSizeBytes);
        FS_HIP(hipFuncSetAttribute((const void *)rank_code_kernel,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, kBinTableBytes));
        if (dev >= 0 && dev < 16)
            configured[dev] = true;
    }
    hipLaunchKernelGGL(rank_code_kernel, dim3(total_blocks), dim3(kBinThreads), kBinTableBytes,
                       stream, d_desc, n_families);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return fail_hip(e, "rank_code_kernel launch");
    return FS_OK;
}

// ------------------------------------------------------------------------------------------------
// traversal over rank tiles
// ------------------------------------------------------------------------------------------------
// A workgroup has T tiles and 16 / T wavefronts per tile, its slots.  The trees in LDS are dealt to the slots, and
// the T wavefronts of a slot (one per tile) walk the slot's trees, wait for each other, put the slot's next
// trees in their place and wait again, on their own: while one slot copies others walk.  A row's running sum
// goes from slot to slot in tree order, through LDS with a counter that says whose turn it is.
// (One chunk of trees for all wavefronts and barriers around walks, sums and copy: a chunk of eight
// trees of depth 10 took 5500 clocks, 3300 of them walks, the rest copying 64 KB into LDS and
// adding up while nothing else ran.  2.1 M rows, 500 such trees: 4.63 ms, so 3.85.)
//
// Two LDS reads a level are a chain of latencies, so what decides is how many walks fit side by side, and what they need
// is room: half of a tree's splits are its last level and half of its words the
// leaves, each read once a walk.  So both stay in memory, a split and its two values in one record: a slot asks for
// its walks' records, replaces its trees, and then takes the last decisions and adds the values up.  A tree of depth
// 10 is 2 KB in LDS then and four tiles have 16 wavefronts of eight walks.  (2.1 M rows of 164 features, 500 trees of
// depth 10, the call: 3.82 ms with splits of all levels in LDS, 12 wavefronts of six walks, so 3.01; half a million rows,
// 300 trees of depth 8 541 us and 476, of depth 9 627 and 527, 200 of depth 11 353 and 272, 100 of depth 12 in 131 072
// rows 198 and 121.  With the leaves in LDS too, as for depth 8 before, 480 instead of 476, and never less.)
//
// No unit is full then, there: vector issue 61 % of the clocks (47 at 72 walks); an LDS instruction every 4.15 clocks, where the
// reads take 2.9 on the mean at the rates measured for them alone (a feature's 2.4; a node's 2.4 in the first six levels,
// 4.2 to 6.7 in the next three); addresses of vector loads 45, their data 59, a cache access every 1.5 clocks.  The records
// are not what it waits for: with those of all walks of a tree at one address the kernel takes 2.63 ms instead of 2.70.
//
// LDS map:  [0, slots * per_slot * tree_bytes)  the slots' trees, each [unused][splits in heap order, 1-based]
//           [tile0 - T*256 - 128, ...)          running sums [tile][lane], then the counters
//           [tile0 + t*Fc*128, ...)             tile t: features 2i, 2i+1 of row l in the word at
//                                               i*256 + 4*l (Fc = F rounded up to even)
// A split word is rank(thr) << 16 | offset of the feature in a tile (i*256 + 2*(f & 1)).

// K trees at once for this lane's row, `depth` levels down to the places A[k].  base[k] = LDS address of tree k; the 1-based heap
// index i lives at A = base + 4*i, and the step i' = 2i + c is taken on the address itself:
// A' = 2A + (4c - base)   (one select between two per-tree constants and one shift-add).
// (Reading both children of a split together with its feature halves the chain of LDS latencies, but two words cost
// the LDS more bank conflicts than one: 4.67 ms instead of 4.51 for 2.1 M rows under 500 trees of depth 10.)
template <int K>
__device__ __forceinline__ void rank_walk(const uint32_t (&base)[K], int depth, uint32_t lane_base, uint32_t (&A)[K])
{
    uint32_t left[K], right[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        A[k] = base[k] + 4u;
        left[k] = 0u - base[k];
        right[k] = 4u - base[k];
        // keep the two constants as they are: the compiler would otherwise fold the select
        // into select(0,4) - base and spend two more instructions per visit
        asm volatile("" : "+v"(left[k]), "+v"(right[k]));
    }
    for (int l = 0; l < depth; ++l) {
        uint32_t nd[K], x[K];
#pragma unroll
        for (int k = 0; k < K; ++k)
            nd[k] = lds_u(A[k]);
#pragma unroll
        for (int k = 0; k < K; ++k)
            x[k] = lds_u16((nd[k] & 0xFFFFu) + lane_base);
#pragma unroll
        for (int k = 0; k < K; ++k)
            A[k] = (A[k] << 1) + ((x[k] < (nd[k] >> 16)) ? left[k] : right[k]);
    }
}

constexpr int kRankThreads = 64 * kRankWaves;
// 16-byte loads in flight per thread for what the direct loads leave of the tiles.  (That is fewer than 64 pieces, one of a
// thread; but with a single guarded copy instead calls of 20 to 50 us measured up to 2 % more, of 16 384 rows of 60
// features under 500 trees of depth 9 34.7 us and 35.3, and no call less.)
constexpr int kRankTileBatch = 11;

// Counters in LDS that only grow.  Everything in LDS that the wavefront did before count_up() is visible to who
// saw the count: LDS operations of a wavefront are carried out in order, and what it read has arrived.
static __device__ __forceinline__ void count_up(uint32_t counter, int lane)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (lane == 0)
        asm volatile("ds_add_u32 %0, %1" ::"v"(counter), "v"(1u) : "memory");
#else
    (void)counter; (void)lane;
#endif
}

// Until the counter has reached `count`.  (Ends: the wavefronts of a workgroup are all on the compute unit, and
// each counts up as often as it is waited for: see the turns of traverse_rank_kernel.)
static __device__ __forceinline__ void wait_for(uint32_t counter, uint32_t count)
{
#if defined(__HIP_DEVICE_COMPILE__)
    for (;;) {
        uint32_t now;
        asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(now) : "v"(counter) : "memory");
        if ((uint32_t)uniform((int)now) >= count)
            break;
        __builtin_amdgcn_s_sleep(1);
    }
#else
    (void)counter; (void)count;
#endif
}

// REGS: 16-byte registers per thread for a slot's next trees.  (No more than they take: a load of a register too
// many costs as much as one that is needed, eleven for six 25 % of the kernel's time; loads under a
// condition had waits put in front of them, 40 %.)
template <int REGS, bool DUMP>
__global__ void __launch_bounds__(kRankThreads)
traverse_rank_kernel(const FamDesc *__restrict__ descs, int n_families, int first_block)
{
    const int block = first_block + (int)blockIdx.x;
    int lo = 0, hi = n_families - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (descs[mid].rk_block0 <= block)
            lo = mid;
        else
            hi = mid - 1;
    }
    const FamDesc &d = descs[lo];
    const int tid = threadIdx.x;
    const int wave = uniform(tid >> 6), lane = tid & 63;
    const int T = d.rk.tiles;                   // tiles per workgroup
    const int n_slots = d.rk.slots;             // kRankWaves / T or fewer
    const int my_slot = wave / T, my_tile = wave - my_slot * T;
    const int n_tiles = row_tiles(d.n_rows);
    const int tile_first = (block - d.rk_block0) * T;
    const int tiles_here = min(T, n_tiles - tile_first);
    const int Fc = rank_tile_cols(d.n_features);
    const uint32_t tile_bytes = (uint32_t)Fc * 128u;
    const uint32_t tile0 = (uint32_t)d.rk.tile0;
    const uint32_t lane_base = tile0 + (uint32_t)my_tile * tile_bytes + 4u * (uint32_t)lane;
    const uint32_t tree_bytes = (uint32_t)d.rk_tree_bytes;
    const int per_slot = d.rk.per_slot;
    const int n_trees = d.n_trees, depth = d.rk_depth;
    const int n_turns = (n_trees + per_slot - 1) / per_slot;     // turn q: trees [q, q + 1) * per_slot, slot q % n_slots
    const uint32_t sums = tile0 - (uint32_t)T * 256u - 128u, counters = tile0 - 128u;
    const uint32_t my_sum = sums + 256u * (uint32_t)my_tile + 4u * (uint32_t)lane;
    const uint32_t turn_at = counters + 4u * (uint32_t)my_tile;            // turns whose values the sum holds
    const uint32_t slot_at = counters + 64u + 4u * (uint32_t)my_slot;      // how often wavefronts of the slot came by
    // tree_bytes is a multiple of 16, so every tree starts 16-byte aligned
    auto image = FS_GLOBAL(const u32x4, d.rk_nodes);
    // (the records of a tree's last splits, by heap index)
    const int last_bytes = (int)sizeof(RankLast) << (depth - 1);    // of a tree
    auto last_splits = FS_GLOBAL(const uint8_t, d.rk_nodes) + (int64_t)n_trees * tree_bytes - last_bytes;
    const int tree16 = (int)(tree_bytes >> 4);
    // The first trees and the tiles go straight from memory to LDS, 1 KB per wavefront-wide
    // load; what is left of each (fewer than 64 pieces) goes through registers.
    const int first16 = min(n_slots * per_slot, n_trees) * tree16;
    const int first_rest = lds_fill_direct(image, 0u, first16, wave, kRankWaves, lane) + tid;
    // ---- rank tiles: consecutive tiles are one contiguous run ----
    {
        auto src = FS_GLOBAL(const u32x4, d.ranks + (int64_t)tile_first * Fc * 64);
        const int per_tile = Fc * 8;                       // 16-byte pieces per tile
        const int n16 = tiles_here * per_tile;
        const int done = lds_fill_direct(src, tile0, n16, wave, kRankWaves, lane);
        for (int base = done + tid; base < n16; base += kRankTileBatch * kRankThreads) {
            u32x4 t4[kRankTileBatch];
#pragma unroll
            for (int q = 0; q < kRankTileBatch; ++q)
                t4[q] = src[min(base + q * kRankThreads, n16 - 1)];
#pragma unroll
            for (int q = 0; q < kRankTileBatch; ++q) {
                const int i = base + q * kRankThreads;
                if (i < n16)
                    lds_store_u4(tile0 + 16u * (uint32_t)i, t4[q]);   // tiles are contiguous in LDS too
            }
        }
    }
    if (first_rest < first16)
        lds_store_u4(16u * (uint32_t)first_rest, image[first_rest]);
    if (my_slot == 0)
        lds_store_f(my_sum, d.bias);
    if (tid < 32)
        lds_store_f(counters + 4u * (uint32_t)tid, 0.0f);  // (the bits of zero)
    lds_direct_wait();
    __syncthreads();
    if (my_slot >= n_slots)
        return;

    const int r = (tile_first + my_tile) * 64 + lane;
    const bool active = my_tile < tiles_here;
    const uint32_t region = (uint32_t)my_slot * (uint32_t)per_slot * tree_bytes;
    const int in_slot = my_tile * 64 + lane, slot_threads = T * 64;
    uint16_t *leaf_row = nullptr;
    if (DUMP) {
        if (active && d.leaf_idx && r < d.n_rows)
            leaf_row = d.leaf_idx + (int64_t)r * n_trees;
    }
    uint32_t passed = 0;                                   // what the slot's counter has to reach
    for (int q = my_slot; q < n_turns; q += n_slots) {
        const int n = min(per_slot, n_trees - q * per_slot);
        // the slot's next trees: global -> registers
        const int q_next = q + n_slots;
        const int n16 = q_next < n_turns ? min(per_slot, n_trees - q_next * per_slot) * tree16 : 0;
        auto src = image + (int64_t)q_next * per_slot * tree16;
        u32x4 pf[REGS];
        if (n16 > 0) {
#pragma unroll
            for (int j = 0; j < REGS; ++j)
                pf[j] = src[min(in_slot + j * slot_threads, n16 - 1)];
        }
        RankLast kept[kRankMostTrees];                     // last splits, from memory
        uint32_t kept_at[DUMP ? kRankMostTrees : 1];
        auto dump = [&](int k, uint32_t heap) {
            if (DUMP && leaf_row) {
                auto ids = FS_GLOBAL(const uint16_t, d.rk_ids + ((int64_t)q * per_slot << (depth + 1)));
                FS_GLOBAL(uint16_t, leaf_row + q * per_slot)[k] = ids[((uint32_t)k << (depth + 1)) + heap];
            }
        };
        auto add_up = [&](auto trees, const float *v) {
            wait_for(turn_at, (uint32_t)q);
            float acc = lds_f(my_sum);
#pragma unroll
            for (int k = 0; k < decltype(trees)::value; ++k)
                acc = acc + v[k];
            if (q + 1 < n_turns) {
                lds_store_f(my_sum, acc);
                count_up(turn_at, lane);
            } else if (r < d.n_rows) {
                FS_GLOBAL(float, d.row_score)[r] = acc;
            }
        };
        auto walk = [&](auto trees) {
            constexpr int K = decltype(trees)::value;
            uint32_t base[K], at[K];
#pragma unroll
            for (int k = 0; k < K; ++k)
                base[k] = region + (uint32_t)k * tree_bytes;
            rank_walk<K>(base, depth - 1, lane_base, at);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                auto tree = last_splits + (int64_t)(q * per_slot + k) * last_bytes;
                auto from = FS_GLOBAL(const RankLast, tree + 3u * (at[k] - base[k]));
                kept[k].split = from->split;
                kept[k].left = from->left;
                kept[k].right = from->right;
                if (DUMP)
                    kept_at[DUMP ? k : 0] = (at[k] - base[k]) >> 2;
            }
            if (n16 > 0)
                count_up(slot_at, lane);                   // the trees have been read
        };
        auto finish = [&](auto trees) {                    // the last splits, then the sum
            constexpr int K = decltype(trees)::value;
            uint32_t x[K];
            float v[K];
#pragma unroll
            for (int k = 0; k < K; ++k)
                x[k] = lds_u16((kept[k].split & 0xFFFFu) + lane_base);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const bool left = x[k] < (kept[k].split >> 16);
                v[k] = left ? kept[k].left : kept[k].right;
                dump(k, 2u * kept_at[DUMP ? k : 0] + (left ? 0u : 1u));
            }
            add_up(trees, v);
        };
        auto for_trees = [&](auto what) {
            switch (n) {
            case 8: what(RankInt<8>()); break;
            case 7: what(RankInt<7>()); break;
            case 6: what(RankInt<6>()); break;
            case 5: what(RankInt<5>()); break;
            case 4: what(RankInt<4>()); break;
            case 3: what(RankInt<3>()); break;
            case 2: what(RankInt<2>()); break;
            default: what(RankInt<1>());
            }
        };
        if (active)
            for_trees(walk);
        else if (n16 > 0)
            count_up(slot_at, lane);
        if (n16 > 0) {
            passed += (uint32_t)T;
            wait_for(slot_at, passed);
#pragma unroll
            for (int j = 0; j < REGS; ++j) {
                const int i = in_slot + j * slot_threads;
                if (i < n16)
                    lds_store_u4(region + 16u * (uint32_t)i, pf[j]);
            }
            for (int i = in_slot + REGS * slot_threads; i < n16; i += slot_threads)   // trees larger than that
                lds_store_u4(region + 16u * (uint32_t)i, src[i]);
            count_up(slot_at, lane);
            passed += (uint32_t)T;
        }
        if (active)
            for_trees(finish);
        if (n16 > 0)
            wait_for(slot_at, passed);                 // the next trees are there
    }
    // (no trees: the row's score is the bias)
    if (n_turns == 0 && my_slot == 0 && active && r < d.n_rows)
        FS_GLOBAL(float, d.row_score)[r] = d.bias;
}

template <int REGS>
static int launch_rank_regs(const FamDesc *d_desc, int n_families, int total_blocks, bool dump, hipStream_t stream)
{
    static bool configured[16][2] = {};
    int dev = 0;
    FS_HIP(hipGetDevice(&dev));
    // (leaf ids: two registers less, with eight some go to scratch memory; 65 536 rows, 60 trees of depth 12, 58.1 us either way)
    constexpr int kDumpRegs = REGS < 6 ? REGS : 6;
    auto kernel = dump ? traverse_rank_kernel<kDumpRegs, true> : traverse_rank_kernel<REGS, false>;
    if (dev < 0 || dev >= 16 || !configured[dev][dump ? 1 : 0]) {
        hipFuncAttributes attr;
        FS_HIP(hipFuncGetAttributes(&attr, (const void *)kernel));
        if (attr.sharedSizeBytes != 0)
            return fail(FS_EDEVICE, "traverse_rank_kernel was built with %zu bytes of static LDS",
                        (size_t)attr.sharedSizeBytes);
        FS_HIP(hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kRankLdsBytes));
        if (dev >= 0 && dev < 16)
            configured[dev][dump ? 1 : 0] = true;
    }
    constexpr int kMostBlocks = (int)((((int64_t)1 << 32) - 1) / kRankThreads);      // of a launch
    for (int first = 0; first < total_blocks; first += kMostBlocks) {
        const int n = std::min(total_blocks - first, kMostBlocks);
        hipLaunchKernelGGL(kernel, dim3(n), dim3(kRankThreads), kRankLdsBytes, stream, d_desc, n_families, first);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return fail_hip(e, "traverse_rank_kernel launch");
    }
    return FS_OK;
}

int launch_traverse_rank(const FamDesc *d_desc, int n_families, int total_blocks, int regs, bool dump, hipStream_t stream)
{
    if (regs <= 3)
        return launch_rank_regs<3>(d_desc, n_families, total_blocks, dump, stream);
    if (regs <= 4)
        return launch_rank_regs<4>(d_desc, n_families, total_blocks, dump, stream);
    if (regs <= 6)
        return launch_rank_regs<6>(d_desc, n_families, total_blocks, dump, stream);
    return launch_rank_regs<8>(d_desc, n_families, total_blocks, dump, stream);
}

}  // namespace fs
