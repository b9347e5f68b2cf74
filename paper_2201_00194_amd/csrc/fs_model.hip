// fs_model_create / fs_model_destroy: validation of the caller's ensemble and packing into
// the device formats.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <future>
#include <memory>
#include <new>
#include <system_error>
#include <utility>
#include <vector>

#include "fs_forms.h"
#include "fs_internal.h"
#include "fs_treelet_pack.h"

using namespace fs;

namespace {

// What the LDS-staged format needs to know of a tree before its nodes are written.
struct TreeSize {
    int32_t nodes;                   // on the paths from the root
    int32_t bytes;
    int32_t depth;
};

// Size of a tree whose nodes share children: every path to a node counts.  False if it has more nodes
// than the caller's array, as it may unfold without bound.
bool unfolded_size(const int32_t *sf, const int32_t *left, const int32_t *right, int32_t sz, TreeSize *out)
{
    std::vector<std::pair<int32_t, int32_t>> todo(1, {0, 0});    // node, level; breadth first
    out->depth = 0;
    for (size_t i = 0; i < todo.size(); ++i) {
        const int32_t n = todo[i].first, level = todo[i].second;
        if (sf[n] < 0)
            continue;
        todo.push_back({left[n], level + 1});
        todo.push_back({right[n], level + 1});
        out->depth = std::max(out->depth, level + 1);
        if (todo.size() > (size_t)sz)
            return false;
    }
    out->nodes = (int32_t)todo.size();
    return true;
}

// A tree of the LDS-staged format at byte `base` of a chunk image, breadth first, so that the two children of
// a node are next to each other; `ids` = the caller's local id per 4-byte slot of the chunk.  In compact
// chunks the splits (8 bytes) come first, then the leaves (4 bytes); the tree is perfect, so breadth
// first has them in that order.  `order`: room for the tree's nodes.
void write_tree(const int32_t *sf, const float *thr, const int32_t *left, const int32_t *right,
                const float *val, const TreeSize &ts, int n_features, bool compact, uint32_t base,
                uint8_t *image, uint16_t *ids, int32_t *order)
{
    const uint32_t n = (uint32_t)ts.nodes, n_int = compact ? n / 2 : n;
    const uint32_t nan_col = (uint32_t)n_features * 256u;
    uint32_t *words = (uint32_t *)(image + base);
    uint16_t *slots = ids + base / 4;
    uint32_t next = 1;                               // position of the next split's left child
    order[0] = 0;
    for (uint32_t i = 0; i < n; ++i) {
        const int32_t o = order[i];
        const uint16_t id = (uint16_t)o;
        if (sf[o] >= 0) {
            order[next] = left[o];
            order[next + 1] = right[o];
            const uint32_t child = next < n_int ? 8u * next : 8u * n_int + 4u * (next - n_int);
            next += 2;
            memcpy(&words[2 * i], &thr[o], 4);
            words[2 * i + 1] = (((uint32_t)sf[o] * 256u) << 16) | ((child + base) & 0xFFFFu);
            slots[2 * i] = slots[2 * i + 1] = id;
        } else if (compact) {
            memcpy(&words[n_int + i], &val[o], 4);
            slots[n_int + i] = id;
        } else {
            memcpy(&words[2 * i], &val[o], 4);
            // own offset - 8; the tree base is at least 8, so this never underflows
            words[2 * i + 1] = (nan_col << 16) | ((8u * i - 8u + base) & 0xFFFFu);
            slots[2 * i] = slots[2 * i + 1] = id;
        }
    }
}

// Largest chunk image: node offsets are 16 bits, and the kernel stages the next chunk in
// kPrefetchRegs 16-byte registers per thread.
// How many trees a chunk should get.  The wavefronts that share a tile (`share` of them) split a
// chunk's trees into runs of at most 8 and walk a run's trees side by side, so a chunk costs a
// fixed part (copy, barriers, ordered sum), a part per run of its busiest wavefront (the
// dependent LDS reads of one walk) and a part per tree of that wavefront.  Weights fitted to
// measurements, in units of one chunk with one run of few trees: 0.73 fixed, 0.27 per run,
// 0.175 per tree -- e.g. 25 trees over 3 wavefronts are two runs each where 24 are one.  Two
// plans are priced: equal chunks, and chunks that are a multiple of `share` x 8 or of `share`
// with the remainder in a last short chunk; the second is taken if it is clearly cheaper.
// Returns the trees per chunk (`fit` = how many fit in LDS).
static int chunk_tree_target(int n_trees, int fit, int share)
{
    auto cost = [share](int n) {
        const int groups = share * ((n + 8 * share - 1) / (8 * share));
        const int runs = groups / share, per = (n + groups - 1) / groups;
        return 0.73 + runs * (0.27 + 0.175 * per);
    };
    if (fit < 1) fit = 1;
    const int even_chunks = (n_trees + fit - 1) / fit;
    const int even = (n_trees + even_chunks - 1) / even_chunks;
    double best_cost = even_chunks * cost(even);
    int best = even;
    const int step = fit >= 8 * share ? 8 * share : share;
    const int whole = fit / step * step;
    if (whole >= step) {
        const int full = n_trees / whole, rest = n_trees - full * whole;
        const double c = full * cost(whole) + (rest ? cost(rest) : 0.0);
        if (c < 0.95 * best_cost) {
            best_cost = c;
            best = whole;
        }
    }
    return best;
}

// ---- chunk plan of the LDS-staged format --------------------------------------------------------
// The wavefronts that share a tile (`share` of them) split a chunk's trees; every wavefront
// walks its trees in runs of at most 8, side by side, a run to the depth of its deepest tree.
// Trees are therefore sorted by depth and cut into runs of similar depth (the cheapest cut of
// the sorted list into runs no longer than an even split would make them), and the runs are
// dealt out most expensive first, each to the wavefront with the least work so far.  Cost in the
// planner's units (weights fitted to measurements on depth-8 trees: one chunk with one run of few
// trees = 1): a chunk costs 0.73 (copy, barriers, ordered sum) + the work of its busiest
// wavefront, a run (0.034 + 0.022 x trees of the run) x (levels of the run + 1).
struct RunPlan {
    int first, count, depth;         // walk-order entries [first, first + count)
};
struct SlotPlan {
    std::vector<int> order;          // trees of the chunk (indices relative to it) in walk order
    std::vector<RunPlan> runs;       // in walk order: the runs of slot 0, then of slot 1, ...
    int slot_start[17];              // slot s walks runs [slot_start[s], slot_start[s + 1])
    double cost;
};

static double run_cost(int trees, int levels) { return (0.034 + 0.022 * trees) * (levels + 1); }

// `by_depth`: the chunk's trees (relative indices) sorted by depth, deepest first.
static void deal_trees(const std::vector<int> &by_depth, const int *depth, int share, SlotPlan *out)
{
    const int n = (int)by_depth.size();
    const int rounds = (n + 8 * share - 1) / (8 * share);
    int cap = (n + share * rounds - 1) / (share * rounds);
    if (cap > 8) cap = 8;
    if (cap < 1) cap = 1;
    struct Piece { int first, count; double cost; };
    std::vector<Piece> pieces;
    std::vector<int> list;           // the trees in the order the pieces index
    // Plain plan: the trees in their own order, share x rounds runs whose sizes differ by at most
    // one, every run to the depth of its deepest tree.
    long plain_levels = 0;
    {
        const int n_runs = share * rounds, base = n / n_runs, rem = n - base * n_runs;
        for (int j = 0, at = 0; j < n_runs; ++j) {
            const int cnt = base + (j < rem ? 1 : 0);
            int d = 0;
            for (int k = 0; k < cnt; ++k)
                d = std::max(d, depth[at + k]);
            plain_levels += (long)cnt * d;
            at += cnt;
        }
    }
    // Sorted plan: cheapest cut of the depth-sorted list into runs of at most `cap`
    std::vector<double> best((size_t)n + 1, 1e300);
    std::vector<int> from((size_t)n + 1, 0);
    best[0] = 0.0;
    for (int i = 0; i < n; ++i)
        for (int c = 1; c <= cap && i + c <= n; ++c) {
            const double v = best[(size_t)i] + run_cost(c, depth[by_depth[(size_t)i]]);
            if (v < best[(size_t)(i + c)] - 1e-12) {
                best[(size_t)(i + c)] = v;
                from[(size_t)(i + c)] = i;
            }
        }
    long sorted_levels = 0;
    for (int j = n; j > 0; j = from[(size_t)j]) {
        pieces.push_back({from[(size_t)j], j - from[(size_t)j],
                          run_cost(j - from[(size_t)j], depth[by_depth[(size_t)from[(size_t)j]]])});
        sorted_levels += (long)(j - from[(size_t)j]) * depth[by_depth[(size_t)from[(size_t)j]]];
    }
    // Sorting pays when it takes a tenth of the walked levels away (measured: with fewer shallow
    // trees the uneven wavefronts it leaves cost what the skipped levels save).
    const bool sorted = 10 * sorted_levels <= 9 * plain_levels;
    if (sorted) {
        list = by_depth;
        std::reverse(pieces.begin(), pieces.end());  // deepest (most expensive per tree) first
        std::stable_sort(pieces.begin(), pieces.end(), [](const Piece &x, const Piece &y) { return x.cost > y.cost; });
    } else {
        pieces.clear();
        list.resize((size_t)n);
        for (int j = 0; j < n; ++j)
            list[(size_t)j] = j;
        const int n_runs = share * rounds, base = n / n_runs, rem = n - base * n_runs;
        for (int j = 0, at = 0; j < n_runs; ++j) {
            const int cnt = base + (j < rem ? 1 : 0);
            if (cnt == 0)
                continue;
            // the kernel walks a run to the depth of its FIRST tree: put the deepest first
            int deepest = at;
            for (int k = 1; k < cnt; ++k)
                if (depth[at + k] > depth[deepest])
                    deepest = at + k;
            std::swap(list[(size_t)at], list[(size_t)deepest]);
            pieces.push_back({at, cnt, run_cost(cnt, depth[list[(size_t)at]])});
            at += cnt;
        }
    }
    std::vector<std::vector<Piece>> bins((size_t)share);
    std::vector<double> load((size_t)share, 0.0);
    if (sorted) {
        for (const Piece &pc : pieces) {
            int to = 0;
            for (int b = 1; b < share; ++b)
                if (load[(size_t)b] < load[(size_t)to] - 1e-12)
                    to = b;
            bins[(size_t)to].push_back(pc);
            load[(size_t)to] += pc.cost;
        }
    } else {
        for (size_t j = 0; j < pieces.size(); ++j) {      // run j to slot j mod share
            bins[j % (size_t)share].push_back(pieces[j]);
            load[j % (size_t)share] += pieces[j].cost;
        }
    }
    out->order.clear();
    out->runs.clear();
    out->cost = 0.0;
    for (int b = 0; b < share; ++b) {
        out->slot_start[b] = (int)out->runs.size();
        for (const Piece &pc : bins[(size_t)b]) {
            out->runs.push_back({(int)out->order.size(), pc.count, depth[list[(size_t)pc.first]]});
            for (int j = 0; j < pc.count; ++j)
                out->order.push_back(list[(size_t)(pc.first + j)]);
        }
        if (load[(size_t)b] > out->cost)
            out->cost = load[(size_t)b];
    }
    for (int b = share; b <= 16; ++b)
        out->slot_start[b] = (int)out->runs.size();
    out->cost += 0.73;
}

size_t chunk_image_limit(int mode)
{
    const size_t by_regs = (size_t)kLdsModeWaves[mode] * 64 * kPrefetchRegs * 16;
    return by_regs < (size_t)kMaxChunkBytes ? by_regs : (size_t)kMaxChunkBytes;
}

// ---- LDS-staged format: which trees go into which chunk --------------------------------------------
struct LdsPlan {
    int mode = 0, tiles = 0;
    bool compact = false;
    std::vector<TreeSize> trees;
    std::vector<int> bounds;         // chunk i holds trees [bounds[i], bounds[i + 1])
    std::vector<SlotPlan> slots;     // per chunk
    float group_us = 0.0f;           // one tile group, estimated
};

// False if the model does not fit the format.
bool plan_lds(int n_features, int n_trees, const TreeShapes &shapes, const int32_t *tree_off, const int32_t *sf,
              const int32_t *left, const int32_t *right, LdsPlan *out)
{
    const int tile_bytes = (n_features + 1) * 256;
    const bool compact = shapes.perfect_depth() >= 0;
    out->compact = compact;
    out->trees.resize((size_t)n_trees);
    size_t max_tree = 0, sum_tree = 0;
    for (int t = 0; t < n_trees; ++t) {
        TreeSize &ts = out->trees[(size_t)t];
        const TreeShapes::Tree &shape = shapes.trees[(size_t)t];
        ts = {shape.n_split + shape.n_leaf, 0, shape.depth};
        const int32_t o = tree_off[t];
        if (!shape.tree && !unfolded_size(sf + o, left + o, right + o, tree_off[t + 1] - o, &ts))
            return false;
        ts.bytes = compact ? 8 * shape.n_split + 4 * shape.n_leaf : 8 * ts.nodes;
        max_tree = std::max(max_tree, (size_t)ts.bytes);
        sum_tree += (size_t)ts.bytes;
    }
    const size_t avg_tree = sum_tree / (size_t)n_trees;
    // Pick the workgroup shape and the number of row tiles per workgroup.  More tiles
    // mean fewer passes of the model through LDS, but less room for trees; what hides
    // LDS latency is the number of independent walks in flight (tiles x trees
    // resident), so that comes first.  The small shape is taken when it still gets 8
    // or more trees into a chunk.
    int best_t = 0, best_score = -1, best_mode = 0;
    size_t best_avail = 0;
    const int forced_tiles = tune(FS_TUNE_LDS_TILES), forced_mode = tune(FS_TUNE_LDS_MODE);
    for (int mode = kLdsModes - 1; mode >= 0 && best_t == 0; --mode) {
        // The half-LDS shape (two workgroups per compute unit) measured no faster on
        // any workload and doubles the model traffic from L2: tuning aid only.
        if (mode == 0 && forced_mode != 1)
            continue;
        if (forced_mode >= 1 && forced_mode <= kLdsModes && mode != forced_mode - 1)
            continue;
        const int max_tiles = mode == 0 ? 1 : kLdsMaxTiles;
        for (int nt = max_tiles; nt >= 1; --nt) {
            if (mode == 1 && forced_tiles >= 1 && forced_tiles <= kLdsMaxTiles && nt != forced_tiles)
                continue;
            const long avail = (long)kLdsModeBytes[mode] - (long)nt * tile_bytes - 64;
            const size_t per_tree_val = (size_t)nt * 256;
            const size_t per_tree_tab = 4;   // a tree word of a run record
            const size_t head = (size_t)(kLdsMaxWaves + 12) * kRunBytes + 16;   // records + padding
            if (avail < (long)(max_tree + head + per_tree_val))
                continue;
            const size_t max_img = chunk_image_limit(mode);
            if (max_img < max_tree + head)
                continue;
            size_t by_chunk = (max_img - head) / (avg_tree + per_tree_tab);
            size_t by_avail = ((size_t)avail - head) / (avg_tree + per_tree_tab + per_tree_val);
            size_t per = by_chunk < by_avail ? by_chunk : by_avail;
            if (per < 1) per = 1;
            if (per > (size_t)kMaxChunkTrees) per = kMaxChunkTrees;
            if (mode == 0 && per < 8 && forced_mode != 1)
                continue;
            int score = nt * (int)per;
            if (score > 64) score = 64;   // measured: beyond ~5 trees per wavefront more
                                          // tiles win, below it more trees per chunk do
            if (score > best_score) {
                best_score = score;
                best_t = nt;
                best_mode = mode;
                best_avail = (size_t)avail;
            }
        }
    }
    if (best_t == 0)
        return false;
    if (tune(FS_TUNE_VERBOSE) > 0)
        fprintf(stderr, "fs_model_create: mode=%d tiles=%d avail=%zu avg_tree=%zu max_tree=%zu compact=%d\n",
                best_mode, best_t, best_avail, avg_tree, max_tree, (int)compact);
    const size_t per_tree_val = (size_t)best_t * 256;
    out->tiles = best_t;
    out->mode = best_mode;
    // Trees per chunk: estimated from the average tree, then balanced over the
    // wavefronts that share a tile (chunk_tree_target); a chunk ends early if its
    // trees are larger than average and the next one does not fit.
    const int share = kLdsModeWaves[best_mode] / best_t;
    const size_t img_limit = chunk_image_limit(best_mode);
    std::vector<int> tdepth((size_t)n_trees);
    for (int t = 0; t < n_trees; ++t)
        tdepth[(size_t)t] = out->trees[(size_t)t].depth;
    // (every tree may need a run record of its own on top of the slots' first records)
    const size_t head0 = (size_t)kLdsMaxWaves * kRunBytes + 16;
    size_t est_per = (best_avail - head0) / (avg_tree + kRunBytes + per_tree_val);
    const size_t est_img = (img_limit - head0) / (avg_tree + kRunBytes);
    if (est_per > est_img) est_per = est_img;
    if (est_per > (size_t)kMaxChunkTrees) est_per = kMaxChunkTrees;
    if (est_per < 1) est_per = 1;
    const int even_cap = chunk_tree_target(n_trees, (int)est_per, share);
    out->bounds.assign(1, 0);
    for (int t = 0; t < n_trees;) {
        int cnt = 0;
        size_t body = 0;
        while (t + cnt < n_trees && cnt < kMaxChunkTrees && cnt < even_cap) {
            const size_t bt = (size_t)out->trees[(size_t)(t + cnt)].bytes;
            // run records in front of the nodes: at most one per slot and one per tree
            const size_t img = ((size_t)(kLdsMaxWaves + cnt + 1) * kRunBytes + body + bt + 15) & ~(size_t)15;
            if (img > img_limit || img + (size_t)(cnt + 1) * per_tree_val > best_avail)
                break;
            body += bt;
            ++cnt;
        }
        t += cnt;                                 // cnt >= 1 by the choice of best_t
        out->bounds.push_back(t);
    }
    out->slots.resize(out->bounds.size() - 1);
    std::vector<int> by_depth;
    for (size_t ci = 0; ci + 1 < out->bounds.size(); ++ci) {
        const int t = out->bounds[ci], cnt = out->bounds[ci + 1] - t;
        by_depth.resize((size_t)cnt);
        for (int j = 0; j < cnt; ++j)
            by_depth[(size_t)j] = j;
        std::stable_sort(by_depth.begin(), by_depth.end(), [&](int x, int y) {
            return tdepth[(size_t)(t + x)] > tdepth[(size_t)(t + y)];
        });
        deal_trees(by_depth, tdepth.data() + t, share, &out->slots[ci]);
        // (the plan's cost is in units of about 1.5 us: 12.1 for 18 us a group of 200 trees of depth 8)
        out->group_us += 1.5f * (float)out->slots[ci].cost;
    }
    return true;
}

void write_lds(const LdsPlan &plan, int n_features, const int32_t *tree_off, const int32_t *sf, const float *thr,
               const int32_t *left, const int32_t *right, const float *val, std::vector<uint8_t> *image,
               std::vector<ChunkHdr> *chunks, std::vector<uint16_t> *slot_ids)
{
    const int share = kLdsModeWaves[plan.mode] / plan.tiles;
    size_t most_nodes = 0;
    for (const TreeSize &ts : plan.trees)
        most_nodes = std::max(most_nodes, (size_t)ts.nodes);
    std::vector<int32_t> order(most_nodes);
    std::vector<int> rec_of;                             // record index of every run
    std::vector<uint32_t> root_at;
    // the images' sizes, so that they are allocated once
    std::vector<size_t> table(plan.slots.size());
    size_t total = 0;
    for (size_t ci = 0; ci < plan.slots.size(); ++ci) {
        const SlotPlan &sp = plan.slots[ci];
        size_t n_rec = kLdsMaxWaves;                     // one per slot first (its first run, or an empty one), then the rest
        for (int b = 0; b < share; ++b)
            if (sp.slot_start[b + 1] > sp.slot_start[b])
                n_rec += (size_t)(sp.slot_start[b + 1] - sp.slot_start[b] - 1);
        table[ci] = (n_rec * kRunBytes + 7) & ~(size_t)7;
        size_t body = 0;
        for (int t = plan.bounds[ci]; t < plan.bounds[ci + 1]; ++t)
            body += (size_t)plan.trees[(size_t)t].bytes;
        ChunkHdr h;
        memset(&h, 0, sizeof(h));
        h.byte_off = (uint32_t)total;
        h.bytes = (uint32_t)((table[ci] + body + 15) & ~(size_t)15);
        h.n_trees = (uint32_t)(plan.bounds[ci + 1] - plan.bounds[ci]);
        h.first_tree = (uint32_t)plan.bounds[ci];
        h.slot_off = (uint32_t)(total / 4);
        chunks->push_back(h);
        total += h.bytes;
    }
    image->assign(total, 0);
    slot_ids->assign(total / 4, 0);
    for (size_t ci = 0; ci < plan.slots.size(); ++ci) {
        const SlotPlan &sp = plan.slots[ci];
        ChunkHdr &h = (*chunks)[ci];
        uint8_t *img = image->data() + h.byte_off;
        uint16_t *ids = slot_ids->data() + h.slot_off;
        size_t pos = table[ci];
        root_at.resize(h.n_trees);
        for (uint32_t j = 0; j < h.n_trees; ++j) {
            const size_t t = h.first_tree + j;
            const TreeSize &ts = plan.trees[t];
            const int32_t o = tree_off[t];
            root_at[j] = (uint32_t)pos;
            write_tree(sf + o, thr + o, left + o, right + o, val + o, ts, n_features, plan.compact, (uint32_t)pos, img,
                       ids, order.data());
            pos += (size_t)ts.bytes;
            h.depth = std::max(h.depth, (uint32_t)ts.depth);
        }
        rec_of.assign(sp.runs.size(), -1);
        int n_rec = kLdsMaxWaves;
        for (int b = 0; b < share; ++b)
            for (int r = sp.slot_start[b]; r < sp.slot_start[b + 1]; ++r)
                rec_of[(size_t)r] = r == sp.slot_start[b] ? b : n_rec++;
        for (int b = 0; b < share; ++b)
            for (int r = sp.slot_start[b]; r < sp.slot_start[b + 1]; ++r) {
                const RunPlan &rp = sp.runs[(size_t)r];
                const int next = r + 1 < sp.slot_start[b + 1] ? rec_of[(size_t)(r + 1)] + 1 : 0;
                uint32_t rec[kRunWords];
                rec[0] = (uint32_t)rp.count | ((uint32_t)next << 4) | ((uint32_t)rp.depth << 16);
                for (int k = 0; k < 8; ++k) {
                    const int j = sp.order[(size_t)(rp.first + (k < rp.count ? k : 0))];
                    rec[1 + k] = root_at[(size_t)j] | ((uint32_t)j << 16);
                }
                memcpy(img + (size_t)rec_of[(size_t)r] * kRunBytes, rec, sizeof(rec));
            }
    }
}

// The bucket of x as the device rounds, truncates and clamps: x * scale is exact in double, so the sum in double rounded
// to float is the fused result unless the rounding to double has made it a tie between two floats, which is noted in
// `tie` or, without that, settled.
inline int rank_bucket(float x, const RankColumn &c, bool *tie)
{
    const double sum = (double)x * (double)c.scale + (double)c.offset;
    uint64_t sum_bits;
    memcpy(&sum_bits, &sum, 8);
    float t = (float)sum;
    const bool is_tie = (sum_bits & 0x1FFFFFFFu) == 0x10000000u;
    if (tie)
        *tie |= is_tie;
    else if (is_tie)
        t = std::fmaf(x, c.scale, c.offset);
    return (int)std::min(t > 0.0f ? t : 0.0f, (float)(c.buckets - 1));
}

// Tables of RankColumn for the rank coder; false where they do not fit or thresholds crowd into few buckets (16 or more
// in one): the bucket and its steps would come near the search tree's, whose reads spread better over the LDS banks.
// The coder's time over 0.5 M rows of 164 features, tree / buckets, us: thresholds of 500 trees of depth 10 175 / 143
// (3 steps), 178 / 150 (4); of 250 of depth 9 154 / 139 (3), 156 / 149 (4), 154 / 155 (5); of 500 of depth 8
// 151 / 138 (3), 155 / 146 (4), 151 / 153 (5).  A call on 2.1 M rows, 500 trees of depth 10: 3.91 / 3.82 ms.
bool bucket_tables(fs_model *m, int n_features, int max_cuts, const std::vector<std::vector<float>> &per,
                   std::vector<float> *tables)
{
    constexpr int kMostSteps = kRankMostSteps, kPast = 1 << (kMostSteps - 1);
    // two buckets a threshold if whole fours of features fit then (the coder searches four at a time), else what is left
    const int keys = (max_cuts + kPast + 3) & ~3;
    int group = kBinTableBytes / (16 + 4 * keys + 4 * max_cuts) & ~3;
    if (group < 4)
        group = 4;
    group = std::min(group, (n_features + 3) & ~3);
    const int B = std::min((kBinTableBytes / group - 16 - 4 * keys) / 2, std::max(4 * max_cuts, 64)) & ~7;
    if (B < std::max(64, max_cuts / 2) || B > 65536)
        return false;
    auto find_buckets = [&](const std::vector<float> &v, const RankColumn &c, std::vector<int> &out) {
        out.resize(v.size());
        bool ties = false;
        for (size_t i = 0; i < v.size(); ++i)
            out[i] = rank_bucket(v[i], c, &ties);
        for (size_t i = 0; i < v.size() && ties; ++i)
            out[i] = rank_bucket(v[i], c, nullptr);
    };
    std::vector<RankColumn> cols((size_t)n_features);
    std::vector<std::vector<int>> bucket((size_t)n_features);
    std::vector<int> tried;
    int most_load = 0;
    for (int f = 0; f < n_features; ++f) {
        const std::vector<float> &v = per[(size_t)f];
        int lo = 0, hi = (int)v.size() - 1, best_load = (int)v.size();
        while (lo < hi && std::isinf(v[(size_t)lo])) ++lo;
        while (hi > lo && std::isinf(v[(size_t)hi])) --hi;
        RankColumn best = {0.0f, 0.0f, B, 0};             // one bucket for all
        bucket[(size_t)f].assign(v.size(), 0);
        // the buckets cover all finite thresholds, or all but the lowest (an exact zero far below the rest) or highest
        for (int trial = 0; trial < 4 && best_load > 7; ++trial) {
            const int a = std::min(lo + (trial & 1), hi), b = std::max(hi - (trial >> 1), a);
            const double span = (double)v[(size_t)b] - (double)v[(size_t)a];
            if (!(span > 0.0))
                continue;
            const double s = (B - 2.0) / span, o = 1.0 - (double)v[(size_t)a] * s;
            if (!(s < 3e38 && s > 1e-37 && std::fabs(o) < 3e38))
                continue;
            const RankColumn c = {(float)s, (float)o, B, 0};
            find_buckets(v, c, tried);
            int load = 0, run = 0, prev = -1;
            for (const int bk : tried) {
                run = bk == prev ? run + 1 : 1;
                prev = bk;
                load = std::max(load, run);
            }
            if (load < best_load) {
                best_load = load;
                best = c;
                bucket[(size_t)f].swap(tried);
            }
        }
        most_load = std::max(most_load, best_load);
        cols[(size_t)f] = best;
    }
    int steps = 0;
    while ((1 << steps) - 1 < most_load)
        ++steps;
    if (steps > kMostSteps)
        return false;
    const size_t stride = (size_t)(16 + 2 * B + 4 * keys);
    tables->assign(stride / 4 * (size_t)n_features, 0.0f);
    for (int f = 0; f < n_features; ++f) {
        const std::vector<float> &v = per[(size_t)f];
        char *const tab = (char *)tables->data() + stride * (size_t)f;
        cols[(size_t)f].steps = steps;
        memcpy(tab, &cols[(size_t)f], sizeof(RankColumn));
        uint16_t *const below = (uint16_t *)(tab + 16);
        int b = 0;
        for (size_t i = 0; i <= v.size(); ++i) {
            const int end = i < v.size() ? bucket[(size_t)f][i] + 1 : B;
            for (; b < end; ++b)
                below[b] = (uint16_t)i;
        }
        float *const key = (float *)(tab + 16 + 2 * B);
        for (int i = 0; i < keys; ++i)
            key[i] = i < (int)v.size() ? v[(size_t)i] : __builtin_nanf("");
    }
    m->cut_bits = -(int)stride;
    m->bin_group = group;
    return true;
}

}  // namespace

// Workgroups of the walk: what is walked side by side decides (no unit is full), up to eight
// trees a slot, and how full the last round of workgroups is.  0.5 M rows of 164 features, 500 trees of depth 10, us by tiles
// a workgroup: 849 with 4 (128 walks), 896 with 5 (120), 897 with 3 (120), 946 with 6 (96), 963 with 2 (112); 4800 rows: 213
// with 8, 136 with 6, 90 with 4, 59 with 2, 48 with 1.  40 000 rows of 60 features, 300 trees of depth 8: 63, 63, 50, 57, 68,
// 82 and 93 us with 1, 2, 3, 4, 5, 6 and 8: 14 us of coding, and a workgroup takes 3.8 us for all its trees' turns and 7.4 more.
RankShape fs::rank_shape(int n_features, int n_trees, int tree_bytes, int64_t own_tiles, int64_t all_tiles, int forced)
{
    const long tile_bytes = (long)rank_tile_cols(n_features) * 128;
    RankShape best = {0, 0, 0, 0};
    double least = 0.0;
    for (const int nt : {8, 6, 5, 4, 3, 2, 1}) {
        if (forced > 0 ? nt != forced : nt > std::max<int64_t>(own_tiles, 1))
            continue;
        const long avail = (long)kRankLdsBytes - nt * (tile_bytes + 256) - 128;
        const int fit = avail < 0 ? 0 : (int)std::min<long>(avail / tree_bytes, 1024);
        RankShape shape = {0, 0, 0, 0};
        for (int slots = std::min(kRankWaves / nt, fit); slots >= 1; --slots) {
            const int per = std::min(fit / slots, kRankMostTrees);
            if (slots * per > shape.slots * shape.per_slot)
                shape = {nt, slots, per, kRankLdsBytes - nt * (int)tile_bytes};
        }
        if (shape.tiles == 0)
            continue;
        const int at_once = std::max(1, std::min(shape.slots * shape.per_slot, n_trees));
        const int64_t rounds = ((all_tiles + nt - 1) / nt + 255) / 256;
        const double time = (double)rounds * (2.0 + (double)n_trees / at_once);
        if (best.tiles > 0 && time >= least)
            continue;
        least = time;
        // as many trees in every turn as the number of turns needs
        const int turns = std::max(1, (n_trees + shape.slots * shape.per_slot - 1) / (shape.slots * shape.per_slot));
        shape.per_slot = std::max(1, (n_trees + shape.slots * turns - 1) / (shape.slots * turns));
        best = shape;
    }
    return best;
}

namespace {

// Rank-coded image of a model of perfect trees of one depth (see fs_rank.hip): per feature the
// sorted distinct thresholds; per tree the splits, word i = heap node i (1-based) as
// rank << 16 | offset of the feature in a rank tile, without the last level; behind those of all trees the last level's
// splits with their leaves' values (RankLast); plus the caller's node id per heap node.
void build_rank_format(fs_model *m, int n_features, int n_trees, int depth, const int32_t *tree_off,
                       const int32_t *sf, const float *thr, const int32_t *left,
                       const int32_t *right, const float *val, std::vector<uint32_t> *nodes,
                       std::vector<uint16_t> *ids, std::vector<float> *cuts)
{
    // thresholds per feature: -0 joins +0, NaN thresholds never send anything left (rank 0)
    std::vector<std::vector<float>> per((size_t)n_features);
    const int64_t n_nodes = tree_off[n_trees];
    for (int64_t g = 0; g < n_nodes; ++g)
        if (sf[g] >= 0 && thr[g] == thr[g])
            per[(size_t)sf[g]].push_back(thr[g] + 0.0f);
    size_t max_cuts = 0;
    for (int f = 0; f < n_features; ++f) {
        std::vector<float> &v = per[(size_t)f];
        std::sort(v.begin(), v.end());
        v.erase(std::unique(v.begin(), v.end()), v.end());
        if (v.size() > max_cuts) max_cuts = v.size();
    }
    int bits = 2;                                         // stride of 2^bits entries per feature
    while ((((size_t)1 << bits) - 1) < max_cuts)
        ++bits;
    const size_t len = (size_t)1 << bits;
    if (bits > 15 || len * 4 > (size_t)kBinTreeBytes)
        return;                                           // ranks must fit 16 bits and LDS
    m->cut_bits = bits;
    m->bin_group = std::min(kBinTreeBytes / 4 / (int)len, n_features);
    if (!bucket_tables(m, n_features, (int)max_cuts, per, cuts)) {
        // else: per feature the sorted keys, padded with NaN to 2^bits - 1, as an implicit search tree in
        // breadth-first order: node 2^l + k (k-th of level l) holds sorted key (2k+1)*2^(bits-l-1) - 1
        cuts->assign(len * (size_t)n_features, __builtin_nanf(""));
        for (int f = 0; f < n_features; ++f) {
            const std::vector<float> &v = per[(size_t)f];
            float *tab = cuts->data() + (size_t)f * len;
            for (int l = 0; l < bits; ++l)
                for (size_t k = 0; k < ((size_t)1 << l); ++k) {
                    const size_t sorted_idx = (2 * k + 1) * ((size_t)1 << (bits - l - 1)) - 1;
                    if (sorted_idx < v.size())
                        tab[((size_t)1 << l) + k] = v[sorted_idx];
                }
        }
    }

    const size_t tree_bytes = std::max<size_t>(16, (size_t)2 << depth);   // (whole 16-byte pieces)
    m->rk_forced_tiles = tune(FS_TUNE_RANK_TILES);
    if (rank_shape(n_features, n_trees, (int)tree_bytes, 1, 1, m->rk_forced_tiles).tiles == 0)
        return;                                           // (too large: other walks take them)
    const size_t words = (size_t)2 << depth, n_leaves = words / 2, stride = tree_bytes / 4;   // per tree, word 0 unused
    const size_t n_last = n_leaves / 2, last_words = 3;
    nodes->assign((stride + n_last * last_words) * (size_t)n_trees, 0u);
    ids->assign(words * (size_t)n_trees, 0);
    std::vector<int32_t> at(words);                       // caller's node at heap position i
    for (int t = 0; t < n_trees; ++t) {
        const int32_t o = tree_off[t];
        uint32_t *const splits = nodes->data() + (size_t)t * stride;
        uint32_t *const last = nodes->data() + stride * (size_t)n_trees + (size_t)t * n_last * last_words;
        at[1] = 0;
        for (size_t i = 1; i < words; ++i) {
            const int32_t n = at[i];
            if (sf[o + n] >= 0) {
                at[2 * i] = left[o + n];
                at[2 * i + 1] = right[o + n];
                const float th = thr[o + n];
                uint32_t rank = 0;
                if (th == th) {
                    const std::vector<float> &v = per[(size_t)sf[o + n]];
                    auto from = v.begin();
                    if (m->cut_bits < 0) {                // not in a lower bucket
                        const char *tab = (const char *)cuts->data() + (int64_t)-m->cut_bits * sf[o + n];
                        RankColumn c;
                        memcpy(&c, tab, sizeof(c));
                        from += ((const uint16_t *)(tab + sizeof(c)))[rank_bucket(th + 0.0f, c, nullptr)];
                        while (*from < th)
                            ++from;
                    } else {
                        from = std::lower_bound(from, v.end(), th + 0.0f);
                    }
                    rank = 1u + (uint32_t)(from - v.begin());
                }
                (i < n_last ? splits[i] : last[(i - n_last) * last_words]) = (rank << 16) | rank_feature_offset(sf[o + n]);
            } else {
                memcpy(&last[(i / 2 - n_last) * last_words + 1 + (i & 1)], &val[o + n], 4);
            }
            (*ids)[(size_t)t * words + i] = (uint16_t)n;
        }
    }
    m->rank_ok = true;
    m->rk_depth = depth;
    m->rk_tree_bytes = (int32_t)tree_bytes;
    if (tune(FS_TUNE_VERBOSE) > 0)
        fprintf(stderr, "fs_model_create: rank-coded depth=%d max_cuts=%zu\n", depth, max_cuts);
}

void free_device(fs_model *m)
{
    if (m->d_nodes) (void)hipFree(m->d_nodes);
    if (m->d_tree_off) (void)hipFree(m->d_tree_off);
    if (m->d_image) (void)hipFree(m->d_image);               // (the chunks and ids lie behind)
    if (m->d_rk_nodes) (void)hipFree(m->d_rk_nodes);
    if (m->d_rk_ids) (void)hipFree(m->d_rk_ids);
    if (m->d_cuts) (void)hipFree(m->d_cuts);
    if (m->d_tl_data) (void)hipFree(m->d_tl_data);
}

template <typename T>
hipError_t upload(T **dst, const std::vector<T> &src)
{
    *dst = nullptr;
    if (src.empty())
        return hipSuccess;
    hipError_t e = device_malloc((void **)dst, src.size() * sizeof(T));
    if (e != hipSuccess)
        return e;
    return hipMemcpy(*dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice);
}

// One allocation and one copy: [images][chunks][ids].
hipError_t upload_lds(fs_model *m, std::vector<uint8_t> &image, const std::vector<ChunkHdr> &chunks,
                      const std::vector<uint16_t> &slot_ids)
{
    const size_t chunk_at = (image.size() + 255) & ~(size_t)255, chunk_bytes = chunks.size() * sizeof(ChunkHdr);
    const size_t ids_at = (chunk_at + chunk_bytes + 255) & ~(size_t)255, ids_bytes = slot_ids.size() * sizeof(uint16_t);
    image.resize(ids_at + ids_bytes, 0);
    memcpy(&image[chunk_at], chunks.data(), chunk_bytes);
    memcpy(&image[ids_at], slot_ids.data(), ids_bytes);
    const hipError_t e = upload(&m->d_image, image);
    m->d_chunks = (ChunkHdr *)(m->d_image + chunk_at);
    m->d_slot_ids = (uint16_t *)(m->d_image + ids_at);
    return e;
}

// One allocation and one copy: [model][segments][chunks][image][ids][columns and tables per segment],
// the pointers inside set for where it will lie.
hipError_t upload_treelets(const TreeletPlan &tl, void **d_data, TreeletModel **d_model)
{
    size_t total = 0;
    std::vector<std::pair<size_t, size_t>> gaps;     // between the parts
    auto room = [&](size_t bytes) {
        const size_t at = total;
        total = (total + bytes + 255) & ~(size_t)255;
        gaps.push_back({at + bytes, total});
        return at;
    };
    const size_t model_at = room(sizeof(TreeletModel)), seg_at = room(tl.segments.size() * sizeof(TreeletSegment)),
                 chunk_at = room(tl.chunks.size() * sizeof(TreeletChunk)), image_at = room(tl.image.size()),
                 id_at = room(tl.ids.size() * sizeof(uint16_t));
    std::vector<size_t> cols_at, tables_at;
    for (const TreeletSegmentPlan &sp : tl.segments) {
        cols_at.push_back(room(sp.cols.size() * sizeof(TreeletCol)));
        tables_at.push_back(room(sp.tables.size()));
    }
    hipError_t e = device_malloc(d_data, total);
    if (e != hipSuccess)
        return e;
    uint8_t *base = (uint8_t *)*d_data;
    std::unique_ptr<uint8_t[]> host(new uint8_t[total]);
    for (const auto &g : gaps)
        memset(&host[g.first], 0, g.second - g.first);
    TreeletModel tm;
    memset(&tm, 0, sizeof(tm));
    tm.image = base + image_at;
    tm.chunks = (const TreeletChunk *)(base + chunk_at);
    tm.segments = (const TreeletSegment *)(base + seg_at);
    tm.ids = (const uint16_t *)(base + id_at);
    tm.n_segments = (int32_t)tl.segments.size();
    tm.most_cols = tl.most_cols;
    tm.buf_bytes = tl.buf_bytes;
    tm.max_trees = tl.max_trees;
    memcpy(&host[model_at], &tm, sizeof(tm));
    memcpy(&host[chunk_at], tl.chunks.data(), tl.chunks.size() * sizeof(TreeletChunk));
    memcpy(&host[image_at], tl.image.data(), tl.image.size());
    memcpy(&host[id_at], tl.ids.data(), tl.ids.size() * sizeof(uint16_t));
    for (size_t i = 0; i < tl.segments.size(); ++i) {
        const TreeletSegmentPlan &sp = tl.segments[i];
        TreeletSegment g;
        memset(&g, 0, sizeof(g));
        g.cols = (const TreeletCol *)(base + cols_at[i]);
        g.tables = base + tables_at[i];
        g.n_cols = (int32_t)sp.cols.size();
        g.buckets = sp.buckets;
        g.table_stride = sp.table_stride;
        g.first_chunk = sp.first_chunk;
        g.n_chunks = sp.n_chunks;
        memcpy(&host[seg_at + i * sizeof(g)], &g, sizeof(g));
        memcpy(&host[cols_at[i]], sp.cols.data(), sp.cols.size() * sizeof(TreeletCol));
        memcpy(&host[tables_at[i]], sp.tables.data(), sp.tables.size());
    }
    *d_model = (TreeletModel *)(base + model_at);
    return hipMemcpy(base, host.get(), total, hipMemcpyHostToDevice);
}

enum Wins { kNever, kSometimes, kAlways };

// Whether treelets win the calls that a model prepared for both walks may get, by the estimates.
Wins treelet_wins(const fs_model *m)
{
    constexpr int kUnits = 256;
    const double lengths[] = {1, 256, 257, 512, 513, 1024, 1025, 1536, 2048, 4096, 16384};
    double least = HUGE_VAL, most = 0.0;
    for (int rowmajor = 0; rowmajor < (lds_reads_rowmajor(m) ? 2 : 1); ++rowmajor)
        for (double tiles : lengths) {
            const int form = treelet_form((int64_t)tiles, kUnits);
            const double tl = treelet_call_us(form, m->tl_us[rowmajor][form], m->tl_once_us, ceil(tiles / 4), kUnits);
            const double lds = lds_call_us(form, rowmajor != 0, m->lds_group_us, lds_fetches(m, rowmajor != 0),
                                           (double)m->n_features * m->lds_tiles, ceil(tiles / m->lds_tiles), kUnits);
            least = std::min(least, tl / lds);
            most = std::max(most, tl / lds);
        }
    // (row-major rows of an odd number of features, not looked at here, are mostly the treelets')
    return least > 1.0 && lds_reads_rowmajor(m) ? kNever : most < 0.95 ? kAlways : kSometimes;
}

}  // namespace

extern "C" int fs_model_create(fs_model **out, int32_t n_features, int32_t n_trees,
                               const int32_t *tree_off, const int32_t *split_feature,
                               const float *threshold, const int32_t *left,
                               const int32_t *right, const float *value, float bias)
{
    if (!out)
        return fail(FS_EINVAL, "fs_model_create: out is NULL");
    *out = nullptr;
    if (n_features < 1 || n_features > FS_MAX_FEATURES)
        return fail(FS_EINVAL, "fs_model_create: n_features %d outside [1, %d]", n_features,
                    FS_MAX_FEATURES);
    if (n_trees < 0)
        return fail(FS_EINVAL, "fs_model_create: n_trees %d is negative", n_trees);
    if (!tree_off)
        return fail(FS_EINVAL, "fs_model_create: tree_off is NULL");
    if (tree_off[0] != 0)
        return fail(FS_EINVAL, "fs_model_create: tree_off[0] must be 0");
    for (int t = 0; t < n_trees; ++t) {
        int64_t sz = (int64_t)tree_off[t + 1] - tree_off[t];
        if (sz < 1 || sz > FS_MAX_TREE_NODES)
            return fail(FS_EINVAL, "fs_model_create: tree %d has %lld nodes (allowed 1..%d)", t,
                        (long long)sz, FS_MAX_TREE_NODES);
    }
    const int64_t n_nodes = tree_off[n_trees];
    if (n_nodes > 0 && (!split_feature || !threshold || !left || !right || !value))
        return fail(FS_EINVAL, "fs_model_create: a node array is NULL");

    try {
        // ---- validation, and the shapes of the trees on the way ----
        TreeShapes shapes;
        {
            std::vector<int32_t> level((size_t)n_nodes, -1);     // -1: not on a path from the root
            shapes.trees.resize((size_t)n_trees);
            for (int t = 0; t < n_trees; ++t) {
                const int32_t o = tree_off[t];
                const int32_t sz = tree_off[t + 1] - o;
                const int32_t *sf = split_feature + o, *le = left + o, *ri = right + o;
                int32_t *lev = level.data() + o;
                TreeShapes::Tree ts = {0, 0, 0, true, false};
                int32_t shallowest = sz;
                shapes.begin_tree();
                lev[0] = 0;
                for (int32_t n = 0; n < sz; ++n) {
                    const int32_t l = lev[n];
                    if (sf[n] >= 0) {
                        if (sf[n] >= n_features)
                            return fail(FS_EINVAL, "fs_model_create: tree %d node %d splits on feature "
                                        "%d but the model has %d", t, n, sf[n], n_features);
                        if (le[n] <= n || le[n] >= sz || ri[n] <= n || ri[n] >= sz)
                            return fail(FS_EINVAL, "fs_model_create: tree %d node %d has child ids "
                                        "(%d, %d); they must lie in (%d, %d)", t, n, le[n], ri[n],
                                        n, sz);
                        if (l < 0)
                            continue;
                        if (le[n] == ri[n] || lev[le[n]] >= 0 || lev[ri[n]] >= 0)
                            ts.tree = false;             // a shared child
                        ++ts.n_split;
                        shapes.add_split(l);
                        lev[le[n]] = lev[ri[n]] = l + 1;
                    } else if (l >= 0) {
                        ++ts.n_leaf;
                        ts.depth = std::max(ts.depth, l);
                        shallowest = std::min(shallowest, l);
                    }
                }
                ts.perfect = ts.tree && ts.depth == shallowest && ts.depth >= 1 && ts.depth <= 14;
                shapes.trees[(size_t)t] = ts;
                shapes.end_tree(t, n_trees);
            }
        }
        // depth of the trees if all are perfect and of one depth, else -1
        const int perfect_depth = shapes.perfect_depth();

        fs_model *m = new (std::nothrow) fs_model();
        if (!m)
            return fail(FS_ENOMEM, "fs_model_create: host allocation failed");
        memset(m, 0, sizeof(*m));
        m->n_features = n_features;
        m->n_trees = n_trees;
        m->n_nodes = n_nodes;
        m->bias = bias;

        // perfect trees that the rank walk takes; measured: it pays from depth 8 on (3 KB per tree in the
        // 8-byte-node format)
        const bool ranks_pay = n_features <= 511 && tune(FS_TUNE_RANK) != 0 && perfect_depth <= 12 &&
                               perfect_depth >= (tune(FS_TUNE_RANK) == 1 ? 1 : 8);

        // ---- LDS-staged format, of a large model on a thread of its own beside the treelets ----
        // (Models that may take either walk need both: 400 irregular trees of depth 12, 112 000 nodes, take 2256 us one
        // after the other and 1957 side by side; below 50 000 nodes there is less to gain than a thread costs.)
        constexpr int64_t kLdsAheadNodes = 50000;
        struct LdsBuild {
            LdsPlan plan;
            bool ok = false, written = false;
            std::vector<uint8_t> image;
            std::vector<ChunkHdr> chunks;
            std::vector<uint16_t> slot_ids;
        };
        const auto plan_format = [&](LdsBuild *b) {
            b->ok = plan_lds(n_features, n_trees, shapes, tree_off, split_feature, left, right, &b->plan);
        };
        const auto write_format = [&](LdsBuild *b) {
            if (b->ok && !b->written)
                write_lds(b->plan, n_features, tree_off, split_feature, threshold, left, right, value, &b->image,
                          &b->chunks, &b->slot_ids);
            b->written = true;
        };
        LdsBuild lds;
        std::future<void> lds_ahead;                     // (waits in its destructor)
        if (n_features <= 255 && n_trees >= kTreeletMinTrees && n_nodes >= kLdsAheadNodes && !ranks_pay &&
            tune(FS_TUNE_TREELET) < 0) {
            try {
                lds_ahead = std::async(std::launch::async, [&] {
                    plan_format(&lds);
                    write_format(&lds);
                });
            } catch (const std::system_error &) {        // no thread to be had
            }
        }

        // ---- byte-rank treelets ----
        TreeletPlan tl;
        std::vector<uint32_t> rk_nodes;
        std::vector<uint16_t> rk_ids;
        std::vector<float> cuts;
        {
            // overrides of the other forms ask for those forms
            const bool others = tune(FS_TUNE_LDS_TILES) >= 0 || tune(FS_TUNE_LDS_MODE) >= 0 ||
                                tune(FS_TUNE_LDS_GROUPS) >= 0 || tune(FS_TUNE_RANK) == 1;
            const int want = tune(FS_TUNE_TREELET);
            TreeletLimits limits;
            if (want != 1) {
                limits.any_size = false;
                // A model is worth a second form if a treelet launch costs no more clocks than 13.5 per level
                // of the trees and 3 per feature, which is about what the LDS walk takes for full trees; the
                // call decides between the two.  Models whose chunks do not fit half a compute unit's LDS only
                // take treelets where there is no other LDS form.
                if (n_features <= 255) {
                    limits.pair_only = true;
                    limits.cost = 13.5 * (double)n_trees * (double)shapes.max_depth() + 3.0 * (double)n_features;
                }
                // Every segment codes the rows anew, the rank walk codes them once.  The line was drawn with an earlier
                // form of either walk.  As they are now, time of treelets over the rank walk's, 90 models of 36 to 500
                // perfect trees of depth 8, 24 to 250 features, 1 to 8000 tiles, both layouts: below 400 columns in all
                // models that take treelets 0.22 to 1.94, geometric mean 0.65 (63 models; 176 of 862 calls lose more than
                // 2 %, 163 of them of up to 1024 tiles, where the rank walk gained most since), models that the other
                // limits turn down 0.13 to 2.61, mean 0.67 (25 models, 334 calls, 157 lose); from 400 columns 0.99 to
                // 2.35, mean 1.69 (2 models, 26 calls, 24 lose).  No line on the model alone is right for both: long calls and
                // few trees are the treelets', short calls of many trees the rank walk's.
                if (ranks_pay) {
                    limits.cols = kTreeletMostRankCols;
                    limits.ranks = true;
                }
            }
            auto plan = [&] {
                return build_treelets(n_features, n_trees, shapes, tree_off, split_feature, threshold, left, right,
                                      value, limits, &tl);
            };
            const bool treelets = want != 0 && (want == 1 || (!others && n_trees >= kTreeletMinTrees));
            if (treelets)
                m->tl_ok = plan();
            // ---- rank-coded format: deep perfect trees ----
            if (ranks_pay && !m->tl_ok) {
                build_rank_format(m, n_features, n_trees, perfect_depth, tree_off, split_feature, threshold, left,
                                  right, value, &rk_nodes, &rk_ids, &cuts);
                if (!m->rank_ok && limits.cols != INT_MAX && treelets) {
                    limits.cols = INT_MAX;               // more thresholds of a feature than ranks of 16 bits
                    limits.ranks = false;
                    m->tl_ok = plan();
                }
            }
            m->tl_pair = tl.pair_ok;
            m->tl_cols = tl.most_cols;
            memcpy(m->tl_us, tl.us, sizeof(m->tl_us));
            m->tl_once_us = tl.once_us;
            if (m->tl_ok && tune(FS_TUNE_VERBOSE) > 0)
                fprintf(stderr, "fs_model_create: treelets, %zu segments of up to %d columns, %zu chunks of at most %d "
                        "trees and %d bytes%s, about %.0f clocks per tile\n", tl.segments.size(), m->tl_cols,
                        tl.chunks.size(), tl.max_trees, tl.buf_bytes, tl.pair_ok ? "" : " (whole LDS)", tl.cost);
        }

        // ---- the LDS-staged format, if it is needed ----
        // beside treelets unless they win (or lose) every call; not where treelets were asked for, nor beside
        // those of perfect trees that the rank walk would take, which win
        const bool planned = lds_ahead.valid();
        if (planned)
            lds_ahead.get();
        if (n_trees > 0 && n_features <= 255 && !m->rank_ok &&
            !(m->tl_ok && (tune(FS_TUNE_TREELET) == 1 || ranks_pay))) {
            if (!planned)
                plan_format(&lds);
            m->lds_ok = lds.ok;
            if (m->lds_ok) {
                m->compact = lds.plan.compact;
                m->lds_tiles = lds.plan.tiles;
                m->lds_mode = lds.plan.mode;
                m->lds_group_us = lds.plan.group_us;
                m->lds_tile0 = kLdsModeBytes[lds.plan.mode] - lds.plan.tiles * (n_features + 1) * 256;
                if (m->tl_ok) {
                    const Wins wins = treelet_wins(m);
                    m->lds_ok = wins != kAlways;
                    m->tl_ok = wins != kNever;
                }
            }
            if (m->lds_ok) {
                write_format(&lds);
                if (tune(FS_TUNE_VERBOSE) > 0) {
                    fprintf(stderr, "fs_model_create: %zu chunks, trees per chunk:", lds.chunks.size());
                    for (const ChunkHdr &c : lds.chunks)
                        fprintf(stderr, " %u", c.n_trees);
                    fprintf(stderr, "\n");
                }
                m->n_chunks = (int32_t)lds.chunks.size();
                m->image_bytes = lds.image.size();
            }
        }

        // ---- flat format: what the global-memory kernel walks, for models without another form ----
        std::vector<GNode> nodes;
        if (!m->tl_ok && !m->lds_ok && !m->rank_ok) {
            nodes.resize((size_t)n_nodes);
            for (int t = 0; t < n_trees; ++t) {
                const int32_t o = tree_off[t];
                for (int32_t g = o; g < tree_off[t + 1]; ++g) {
                    GNode &nd = nodes[(size_t)g];
                    if (split_feature[g] < 0) {
                        memcpy(&nd.x, &value[g], 4);
                        nd.y = -1;
                        nd.z = nd.w = g;
                    } else {
                        memcpy(&nd.x, &threshold[g], 4);
                        nd.y = split_feature[g];
                        nd.z = o + left[g];
                        nd.w = o + right[g];
                    }
                }
            }
        }

        hipError_t e = hipGetDevice(&m->device);
        if (e == hipSuccess && !m->tl_ok && !m->lds_ok && !m->rank_ok) {
            std::vector<int32_t> toff(tree_off, tree_off + n_trees + 1);
            e = upload(&m->d_tree_off, toff);
        }
        if (e == hipSuccess) e = upload(&m->d_nodes, nodes);
        if (e == hipSuccess && m->lds_ok)
            e = upload_lds(m, lds.image, lds.chunks, lds.slot_ids);
        if (e == hipSuccess && m->rank_ok) {
            e = upload(&m->d_rk_nodes, rk_nodes);
            if (e == hipSuccess) e = upload(&m->d_rk_ids, rk_ids);
            if (e == hipSuccess) e = upload(&m->d_cuts, cuts);
        }
        if (e == hipSuccess && m->tl_ok)
            e = upload_treelets(tl, &m->d_tl_data, &m->d_tl);
        if (e != hipSuccess) {
            free_device(m);
            delete m;
            return fail_hip(e, "fs_model_create: device upload");
        }
        *out = m;
        return FS_OK;
    } catch (const std::bad_alloc &) {
        return fail(FS_ENOMEM, "fs_model_create: host allocation failed");
    }
}

extern "C" void fs_model_destroy(fs_model *m)
{
    if (!m)
        return;
    free_device(m);
    delete m;
}
