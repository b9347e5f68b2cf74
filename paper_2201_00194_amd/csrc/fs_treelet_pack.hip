// Builds the byte-rank treelet format (fs_treelet.h) of a model on the host.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <utility>
#include <vector>

#include "fs_internal.h"
#include "fs_treelet_pack.h"

namespace fs {

namespace {

struct Piece { int feature, at, n; };                // thresholds [at, at + n) of the feature

// Columns and tables for B buckets.
void build_columns(const std::vector<Piece> &pieces, const std::vector<float> &cuts,
                   const std::vector<int32_t> &cut_at, int B, TreeletSegmentPlan *out)
{
    auto values = [&](const Piece &pc) { return cuts.data() + cut_at[(size_t)pc.feature] + pc.at; };
    // As the device computes it: one rounding of x * scale + offset, clamped to [0, 1], times B - 1, rounded to the
    // nearest integer (ties to even).  x * scale is exact in double, so the sum in double rounded to float is the
    // fused result unless the rounding to double has made it a tie between two floats; the second product is exact too.
    auto bucket_of = [B](float x, const TreeletCol &c) -> int {
        const double sum = (double)x * (double)c.scale + (double)c.offset;
        uint64_t bits;
        memcpy(&bits, &sum, 8);
        float u = (float)sum;
        if ((bits & 0x1FFFFFFFu) == 0x10000000u)
            u = std::fmaf(x, c.scale, c.offset);
        u = u > 0.0f ? std::min(u, 1.0f) : 0.0f;
        constexpr double kToInt = 6755399441055744.0;        // 1.5 * 2^52: adding it rounds
        return (int)(((double)u * (double)(B - 1) + kToInt) - kToInt);
    };
    out->cols.clear();
    int most_cuts = 0, most_steps = 0;
    std::vector<uint16_t> buckets(pieces.size() * (size_t)kTreeletMaxCuts, 0);
    uint16_t tried[kTreeletMaxCuts];
    for (const Piece &pc : pieces) {
        const float *v = values(pc);
        // The range the buckets cover, downwards: all finite thresholds, or all but the highest or the lowest (an
        // exact zero far below the rest), a little wider or narrower; the fullest bucket decides.
        int lo = 0, hi = pc.n - 1;
        while (lo < hi && std::isinf(v[lo])) ++lo;
        while (hi > lo && std::isinf(v[hi])) --hi;
        TreeletCol best = {pc.feature, 0.0f, 0.0f, 0};
        int best_load = pc.n;                        // one bucket for all
        for (int trial = 0; trial < 8 && best_load > 3; ++trial) {
            const int a = std::min(lo + ((trial >> 1) & 1), hi), b = std::max(hi - (trial & 1), a);
            const double span = (double)v[a] - (double)v[b];
            if (!(span > 0.0))
                continue;
            const double s = -(B - 2.0) / (B - 1.0) * (1.0 - 0.07 * (trial >> 2)) / span, o = 1.0 / (B - 1.0) - (double)v[a] * s;
            if (!(s > -3e38 && s < -1e-37 && std::fabs(o) < 3e38))
                continue;
            const TreeletCol c = {pc.feature, (float)s, (float)o, 0};
            int load = 0, run = 0, prev = -1;
            for (int i = 0; i < pc.n && load < best_load; ++i) {
                const int bk = bucket_of(v[i], c);
                tried[i] = (uint16_t)bk;
                run = bk == prev ? run + 1 : 1;
                prev = bk;
                load = std::max(load, run);
            }
            if (load < best_load) {
                best_load = load;
                best = c;
                memcpy(&buckets[out->cols.size() * (size_t)kTreeletMaxCuts], tried, sizeof(tried[0]) * (size_t)pc.n);
            }
        }
        while ((1 << best.steps) - 1 < best_load)
            ++best.steps;
        out->cols.push_back(best);
        most_cuts = std::max(most_cuts, pc.n);
        most_steps = std::max(most_steps, best.steps);
    }
    // probes go up to 2^(steps - 1) - 1 past the number of thresholds
    const int n_keys = (most_cuts + (1 << std::max(most_steps - 1, 0)) + 3) / 4 * 4;
    out->buckets = B;
    out->table_stride = B + 4 * n_keys;
    out->tables.assign(pieces.size() * (size_t)out->table_stride + kTreeletTablePad, 0);
    for (size_t c = 0; c < pieces.size(); ++c) {
        const float *v = values(pieces[c]);
        const uint16_t *bucket = &buckets[c * (size_t)kTreeletMaxCuts];
        uint8_t *tab = out->tables.data() + c * (size_t)out->table_stride;
        // (higher) thresholds in lower buckets, for every bucket: eight at a time (the last writes run into the keys'
        // place, or the next column's, which are written after)
        int b = 0;
        for (int i = 0; i <= pieces[c].n; ++i) {
            const int end = i < pieces[c].n ? bucket[i] + 1 : B;
            const uint64_t eight = 0x0101010101010101ull * (uint64_t)i;
            for (; b < end; b += 8)
                memcpy(tab + b, &eight, 8);
            b = end;
        }
        float *key = (float *)(tab + B);
        for (int i = 0; i < n_keys; ++i)
            key[i] = i < pieces[c].n ? v[i] : __builtin_nanf("");
    }
}

// Thresholds and columns of a segment's trees.
struct SegmentCuts {
    std::vector<float> cuts;                         // distinct, the highest first, per feature
    std::vector<int32_t> cut_at;
    std::vector<Piece> pieces;
};

// Order of floats as unsigned integers (-0 joins +0).
inline uint32_t ordered(float v)
{
    uint32_t b;
    v = v + 0.0f;
    memcpy(&b, &v, 4);
    return (b & 0x80000000u) ? ~b : b | 0x80000000u;
}

// The float of an ordered() value.
inline float unordered(uint32_t k)
{
    k = (k & 0x80000000u) ? k & 0x7FFFFFFFu : ~k;
    float v;
    memcpy(&v, &k, 4);
    return v;
}

// Sorts n keys by their upper halves; `spare` has room for as many.  Returns where they are, keys or spare.
// First into about n buckets of equal width, as the thresholds of a feature are mostly spread over its
// values, then each bucket (whatever the values are, this is no slower than its sort).
uint64_t *sort_keys(uint64_t *keys, uint64_t *spare, int n)
{
    constexpr int kMost = 1024;
    uint32_t lo = 0xFFFFFFFFu, hi = 0;
    for (int i = 0; i < n; ++i) {
        const uint32_t k = (uint32_t)(keys[i] >> 32);
        lo = std::min(lo, k);
        hi = std::max(hi, k);
    }
    const int buckets = std::min(n, kMost);
    const float low = unordered(lo), scale = (float)buckets / (unordered(hi) - low);
    if (n < 16 || !(scale > 0.0f && scale < 3e38f) || std::isinf(low)) {
        std::sort(keys, keys + n);
        return keys;
    }
    uint32_t at[kMost + 1];
    std::fill(at, at + buckets + 1, 0u);
    // (never decreases with the key: subtraction, product and truncation round monotonically)
    auto bucket_of = [&](uint64_t k) {
        return std::min((int)((unordered((uint32_t)(k >> 32)) - low) * scale), buckets - 1);
    };
    for (int i = 0; i < n; ++i)
        ++at[bucket_of(keys[i]) + 1];
    uint32_t fullest = 0;
    for (int b = 0; b < buckets; ++b) {
        fullest = std::max(fullest, at[b + 1]);
        at[b + 1] += at[b];
    }
    for (int i = 0; i < n; ++i)
        spare[at[bucket_of(keys[i])]++] = keys[i];
    if (fullest > 16)
        for (int b = 0; b < buckets; ++b) {          // at[b] is where bucket b ends now
            const uint32_t from = b ? at[b - 1] : 0;
            if (at[b] - from > 16 && !std::is_sorted(spare + from, spare + at[b]))
                std::sort(spare + from, spare + at[b]);   // (equal thresholds arrive in order)
        }
    for (int i = 1; i < n; ++i) {                    // what is left to move stays inside its bucket
        const uint64_t k = spare[i];
        int j = i;
        for (; j > 0 && spare[j - 1] > k; --j)
            spare[j] = spare[j - 1];
        spare[j] = k;
    }
    return spare;
}

// Sorts the thresholds of n_splits nodes, so many of each feature, by feature, lists the columns and sets word[node] = column << 8 |
// rank of every split (rank 255 for a NaN threshold: it sends nothing left).  False if the trees need more
// columns than a byte names.
bool segment_cuts(int n_features, const int32_t *nodes, size_t n_splits, const std::vector<int32_t> &of_feature,
                  const int32_t *sf, const float *thr, std::vector<uint64_t> &keys, uint16_t *word, SegmentCuts *out)
{
    std::vector<int32_t> at((size_t)n_features + 1, 0), fill((size_t)n_features, 0), nan_nodes;
    int32_t most = 0;
    for (int f = 0; f < n_features; ++f) {           // feature f's keys are [at[f], at[f + 1])
        most = std::max(most, of_feature[(size_t)f]);
        at[(size_t)f + 1] = at[(size_t)f] + of_feature[(size_t)f];
        fill[(size_t)f] = at[(size_t)f];
    }
    keys.resize(n_splits + (size_t)most);
    for (size_t i = 0; i < n_splits; ++i) {
        const int32_t g = nodes[i];
        if (thr[g] == thr[g])
            keys[(size_t)fill[(size_t)sf[g]]++] = ((uint64_t)ordered(thr[g]) << 32) | (uint32_t)g;
        else
            nan_nodes.push_back(g);
    }
    uint64_t *spare = keys.data() + n_splits;
    out->cuts.resize(n_splits);
    out->cut_at.assign((size_t)n_features + 1, 0);
    out->pieces.clear();
    std::vector<int32_t> first_col((size_t)n_features, 0);
    for (int f = 0; f < n_features; ++f) {
        if (at[(size_t)f + 1] == at[(size_t)f])
            continue;
        const int first = (int)out->pieces.size();
        first_col[(size_t)f] = first;
        const int m = fill[(size_t)f] - at[(size_t)f];
        const uint64_t *k = sort_keys(keys.data() + at[(size_t)f], spare, m);
        float *v = out->cuts.data() + at[(size_t)f];
        int n = 0, rank = 0;                         // rank inside the piece
        uint32_t piece = (uint32_t)first - 1, last = 0;
        for (int i = m - 1; i >= 0; --i) {
            const uint32_t key = (uint32_t)(k[i] >> 32);
            if (i == m - 1 || key != last) {
                last = key;
                v[n++] = unordered(key);
                if (++rank > kTreeletMaxCuts || i == m - 1) {
                    rank = 1;
                    ++piece;
                }
            }
            word[(uint32_t)k[i]] = (uint16_t)((piece << 8) | (uint32_t)rank);
        }
        out->cut_at[(size_t)f] = at[(size_t)f];
        int from = 0;
        do {
            out->pieces.push_back({f, from, std::min(kTreeletMaxCuts, n - from)});
            from += kTreeletMaxCuts;
        } while (from < n);
        if (out->pieces.size() > (size_t)kTreeletMaxCols)
            return false;
    }
    for (int32_t g : nan_nodes)
        word[g] = (uint16_t)(first_col[(size_t)sf[g]] << 8 | 255);
    if (out->pieces.empty())                         // single leaves only: one column nobody asks
        out->pieces.push_back({0, 0, 0});
    return true;
}

// Times of a round of workgroups in each form (fs_forms.h says what they were fitted to): per segment
// (launch and barriers), column, batch of columns that a wavefront codes, chunk, step of a chunk's deepest
// walk, and step of all its trees.
void estimate_rounds(int n_features, TreeletPlan *p)
{
    struct Spread { int tiles; double call, segment, col, wide, narrow, chunk, step, tree_step; };
    static const Spread spread[2][kTreeletForms] = {
        {{0, 0, 0, 0, 0, 0, 0, 0, 0},
         {4, 3.6, 4.3, 0.054, 0.1, 0.2, 0.72, 0.05, 0.0177},
         {2, 4.9, 3.8, 0.0217, 0.4, 0.27, 0.544, 0.12, 0.0067},
         {1, 5.3, 2.85, 0.0105, 1.35, 0.49, 0.31, 0.206, 0.0026}},
        {{0, 0, 0, 0, 0, 0, 0, 0, 0},
         {4, 2.8, 4.6, 0.083, 0.0, 0.55, 0.67, 0.051, 0.0173},
         {2, 5.2, 3.7, 0.024, 0.4, 0.52, 0.54, 0.123, 0.0068},
         {1, 5.3, 2.85, 0.0105, 1.35, 0.52, 0.31, 0.206, 0.0026}}};
    // the pair form: a column by how many a wavefront codes at a time (4, 2, 1); row-major more the longer a
    // row is, as fewer of its lines are still in a cache when the next batch asks for them
    static const double pair_col[2][3] = {{0.0862, 0.0861, 0.106}, {0.097, 0.207, 0.236}};
    static const double pair_feature[2][3] = {{0.0, 0.0, 0.0}, {2.2e-4, 5.5e-4, 5.5e-4}};
    static const double pair_chunk[2] = {1.13, 1.09}, pair_tree_step[2] = {0.0317, 0.0284};
    auto kb = [](long bytes) { return (bytes + 1023) / 1024 * 1024; };
    double steps = 0.0, tree_steps = 0.0;
    for (const TreeletChunk &c : p->chunks) {
        steps += c.steps;
        tree_steps += (double)c.n_trees * c.steps;
    }
    // Tables of single columns without a second buffer, where the columns leave no room for one: 0.15 us a column
    // more in launches of a round or two (164 features, 200 columns, 3000 tiles: estimated 269, measured
    // 300 us; row-major 323 and 359), nothing in long ones, whose workgroups are out of step (40 000
    // tiles 2845 and 2730, 3579 and 3387).
    double once = 0.0;
    const double n_chunks = (double)p->chunks.size();
    const long columns = (long)p->most_cols * 256;
    for (int rowmajor = 0; rowmajor < 2; ++rowmajor) {
        double pair = pair_chunk[rowmajor] * n_chunks + pair_tree_step[rowmajor] * tree_steps;
        for (const TreeletSegmentPlan &sp : p->segments) {
            const long room = (long)kTreeletLds - kTreeletSumBytes - columns;
            const int batch = 16 * kb(4L * sp.table_stride) <= room ? 0 : 16 * kb(2L * sp.table_stride) <= room ? 1 : 2;
            if (rowmajor == 0 && 16 * kb(sp.table_stride) > room)
                once += 0.15 * (double)sp.cols.size();
            pair += (pair_col[rowmajor][batch] + pair_feature[rowmajor][batch] * n_features) * (double)sp.cols.size();
        }
        p->us[rowmajor][kTreeletPair] = (float)pair;
        for (int form = kTreeletSpread4; form < kTreeletForms; ++form) {
            const Spread &e = spread[rowmajor][form];
            double us = e.call + e.chunk * n_chunks + e.step * steps + e.tree_step * tree_steps;
            for (const TreeletSegmentPlan &sp : p->segments) {
                const int wide = 16 / e.tiles, narrow = 4 / e.tiles;
                const bool fits = 12 * kb((long)wide * sp.table_stride) + p->buf_bytes <= (long)kTreeletLdsWhole - columns;
                const int cols = (int)sp.cols.size(), at_once = 12 * (fits ? wide : narrow);
                us += e.segment + e.col * cols + (fits ? e.wide : e.narrow) * ((cols + at_once - 1) / at_once);
            }
            p->us[rowmajor][form] = (float)us;
        }
    }
    p->once_us = (float)once;
}

}  // namespace

bool build_treelets(int n_features, int n_trees, const TreeShapes &shape, const int32_t *tree_off,
                    const int32_t *sf, const float *thr, const int32_t *left, const int32_t *right, const float *val,
                    const TreeletLimits &limits, TreeletPlan *out)
{
    if (n_trees < 1)
        return false;
    std::vector<uint8_t> tree_steps((size_t)n_trees);
    for (int t = 0; t < n_trees; ++t) {
        if (!shape.trees[(size_t)t].tree || shape.deep)
            return false;
        tree_steps[(size_t)t] = (uint8_t)shape.steps(t);
    }
    // splits at depth 2*s of trees [a, b)
    auto splits = [&](int s, int a, int b) -> int64_t {
        return shape.sum[s].empty() ? 0 : shape.sum[s][(size_t)b] - shape.sum[s][(size_t)a];
    };
    // bytes of a chunk of trees [a, b) (padded to units) and its step count
    auto chunk_size = [&](int a, int b, int *steps, int *entries, int *values) -> size_t {
        int s = 1;
        for (int t = a; t < b; ++t)
            s = std::max(s, (int)tree_steps[(size_t)t]);
        int64_t e = (b - a + kTreeletUnit - 1) / kTreeletUnit * kTreeletUnit;
        for (int i = 0; i + 1 < s; ++i)
            e += 4 * splits(i, a, b);
        const int64_t v = 4 * splits(s - 1, a, b);
        *steps = s;
        *entries = (int)e;
        *values = (int)(e + v);
        return ((size_t)(8 * e + 4 * (e + v)) + 1023) & ~(size_t)1023;
    };
    int s_, e_, v_;
    // Trees so large that a chunk holds a handful walk no faster here than in the other forms.
    if (!limits.any_size && chunk_size(0, n_trees, &s_, &e_, &v_) / (size_t)n_trees * kTreeletFewTrees > (size_t)kTreeletPairBuf)
        return false;

    // ---- segments: as few as their columns allow, equally long ----
    int n_used = 0;                                                  // features
    std::vector<SegmentCuts> seg_cuts;
    std::vector<uint16_t> word((size_t)tree_off[n_trees]);           // column << 8 | rank of the splits
    {
        // (an ensemble whose splits are many times what the columns hold starts with several segments: no
        // sort of a million thresholds only to see that)
        // The splits, and how many each feature has (at [feature + 1]; leaves count at [0]: no branch that a leaf
        // would upset).
        std::vector<int32_t> nodes((size_t)tree_off[n_trees]), n_splits((size_t)n_features + 1, 0);
        size_t all_splits = 0;
        for (int32_t g = 0; g < tree_off[n_trees]; ++g) {
            nodes[all_splits] = g;
            all_splits += sf[g] >= 0;
            ++n_splits[(size_t)(std::max(sf[g], -1) + 1)];
        }
        n_splits.erase(n_splits.begin());
        for (int32_t n : n_splits)
            n_used += n != 0;
        // what the walk costs at least: every used feature one column, every tree its own steps
        double least = 0.0;
        for (int32_t n : n_splits)
            least += n ? kTreeletColClk : 0.0;
        for (uint8_t n : tree_steps)
            least += kTreeletStepClk * n;
        if (least > limits.cost)
            return false;
        int m = 1;
        for (;; ++m) {                               // assumes that half of the splits are distinct
            int64_t cols = 0;
            for (int f = 0; f < n_features; ++f)
                if (n_splits[(size_t)f])
                    cols += std::max<int64_t>(1, n_splits[(size_t)f] / (2 * (int64_t)m * kTreeletMaxCuts));
            if (cols <= kTreeletMaxCols)
                break;
            if (m >= kTreeletMaxSegments)
                return false;
        }
        std::vector<uint64_t> keys;
        for (;; ++m) {
            if (m > kTreeletMaxSegments)
                return false;
            const int per = ((n_trees + m - 1) / m + 7) / 8 * 8;
            out->segments.clear();
            seg_cuts.clear();
            bool ok = true;
            size_t from = 0, to;                         // splits of the segment
            std::vector<int32_t> mine;
            for (int t = 0; t < n_trees && ok; t += per, from = to) {
                out->segments.emplace_back();
                seg_cuts.emplace_back();
                TreeletSegmentPlan &sp = out->segments.back();
                sp.first_tree = t;
                sp.n_trees = std::min(per, n_trees - t);
                to = all_splits;
                if (per < n_trees) {
                    to = (size_t)(std::lower_bound(nodes.begin() + (long)from, nodes.begin() + (long)all_splits,
                                                   tree_off[t + sp.n_trees]) - nodes.begin());
                    mine.assign((size_t)n_features, 0);
                    for (size_t i = from; i < to; ++i)
                        ++mine[(size_t)sf[nodes[i]]];
                }
                ok = segment_cuts(n_features, nodes.data() + from, to - from, per < n_trees ? mine : n_splits, sf, thr,
                                  keys, word.data(), &seg_cuts.back());
            }
            if (ok)
                break;
            if (per <= 8)
                return false;
        }
    }
    out->most_cols = 0;
    for (const SegmentCuts &c : seg_cuts)
        out->most_cols = std::max(out->most_cols, (int)c.pieces.size());
    int all_cols = 0;
    for (const SegmentCuts &c : seg_cuts)
        all_cols += (int)c.pieces.size();
    if (all_cols > limits.cols)
        return false;

    // ---- bounds of the chunks ----
    // Bounds of the chunks of trees [t0, t1) in buffers of `buf` bytes.  Two wavefronts take a chunk's
    // halves in rounds of kTreeletRound: full rounds if the trees fit, else eights, else fours.
    auto plan = [&](int t0, int t1, size_t buf, std::vector<int> *bounds) -> bool {
        bounds->assign(1, t0);
        int s, e, v;
        auto fits = [&](int t, int cnt) { return chunk_size(t, std::min(t1, t + cnt), &s, &e, &v) <= buf; };
        while (bounds->back() < t1) {
            const int t = bounds->back();
            int cnt = kTreeletMaxTrees;
            while (cnt > 2 * kTreeletRound && !fits(t, cnt))
                cnt -= 2 * kTreeletRound;
            while (cnt > 2 * kTreeletUnit && !fits(t, cnt))
                cnt -= 2 * kTreeletUnit;
            if (!fits(t, cnt))
                cnt = kTreeletUnit;
            if (!fits(t, cnt))
                return false;
            bounds->push_back(std::min(t1, t + cnt));
        }
        return true;
    };
    auto plan_all = [&](size_t buf, std::vector<std::vector<int>> *all) -> bool {
        all->resize(out->segments.size());
        for (size_t i = 0; i < out->segments.size(); ++i)
            if (!plan(out->segments[i].first_tree, out->segments[i].first_tree + out->segments[i].n_trees, buf, &(*all)[i]))
                return false;
        return true;
    };
    auto cost_of = [&](const std::vector<std::vector<int>> &all) {
        int steps, e, v;
        double cost = 0.0;
        for (size_t i = 0; i < all.size(); ++i) {
            cost += kTreeletColClk * (double)seg_cuts[i].pieces.size();
            for (size_t c = 0; c + 1 < all[i].size(); ++c) {
                const int n = (all[i][c + 1] - all[i][c] + kTreeletUnit - 1) / kTreeletUnit * kTreeletUnit;
                (void)chunk_size(all[i][c], all[i][c + 1], &steps, &e, &v);
                cost += kTreeletStepClk * (double)n * steps + kTreeletChunkClk;
            }
        }
        return cost;
    };
    // (before the columns' tables, which are most of what is left to do: a model that would be turned down
    // for this costs its sort of the thresholds and no more)
    std::vector<std::vector<int>> all;
    const long room = (long)kTreeletLds - kTreeletSumBytes - (long)out->most_cols * 256;
    out->pair_ok = plan_all(std::min((size_t)room / 1024 * 1024, (size_t)kTreeletPairBuf), &all);
    if (limits.pair_only && !out->pair_ok)
        return false;
    if (out->pair_ok && cost_of(all) > limits.cost)
        return false;

    // ---- columns ----
    // Buckets of every column: five or more per threshold, so that a bucket of evenly spread thresholds
    // holds three at most (two bisection steps), with few exceptions; less where the tables of the
    // wavefronts would not fit beside the columns.
    const long beside = (long)out->most_cols * 256;
    auto kb = [](long bytes) { return (bytes + 1023) / 1024 * 1024; };
    // (the coder's layouts in fs_treelet.hip: a double-buffered table for each of 8 wavefronts, or a single one
    // beside more columns; four tables for each of 12)
    auto pair_fits = [&](int stride, int halves) { return 8 * halves * kb(stride) <= (long)kTreeletLds - kTreeletSumBytes - beside; };
    auto spread_fits = [&](int stride) { return 12 * kb(4 * stride) <= (long)kTreeletLdsWhole - beside; };
    bool pair_coder = true;
    // Where the rank walk could take the model, single tables only with chunks of eight trees and about one column a
    // feature.  Treelets / rank walk, perfect trees of depth 8, 3800 to 1 M rows: 200 and 220 features, 160 and
    // 230 trees 0.53 to 0.87, mean 0.69; 250 features, room for four trees a chunk, 100 to 230 trees 0.48 to 1.32, mean
    // 0.85; 80 and 100 features of two to three columns each, 160 to 300 trees 0.71 to 1.35, mean 0.92; 24 to 64 features
    // of three and more, 230 and 300 trees 0.78 to 1.60, mean 1.02.
    bool single = true;
    if (limits.ranks && out->pair_ok) {
        single = 4 * all_cols <= 5 * n_used;
        for (const std::vector<int> &b : all)
            single = single && b[1] - b[0] >= std::min(8, b.back() - b[0]);
    }
    for (size_t i = 0; i < out->segments.size();) {
        TreeletSegmentPlan *sp = &out->segments[i];
        int most_cuts = 0, want = 64;
        for (const Piece &pc : seg_cuts[i].pieces)
            most_cuts = std::max(most_cuts, pc.n);
        while (want < 5 * most_cuts && want < 1024)
            want *= 2;
        bool fits = false;
        for (int halves = 2; halves >= (single ? 1 : 2) && !fits; --halves)
            for (int B = want; B >= 64 && !fits; B /= 2) {
                const int least = B + 4 * ((most_cuts + 1 + 3) / 4 * 4);   // of what build_columns makes the stride
                if (!spread_fits(least) || (pair_coder && !pair_fits(least, halves)))
                    continue;
                build_columns(seg_cuts[i].pieces, seg_cuts[i].cuts, seg_cuts[i].cut_at, B, sp);
                fits = spread_fits(sp->table_stride) && (pair_fits(sp->table_stride, halves) || !pair_coder);
            }
        if (fits) {
            ++i;
        } else if (limits.pair_only) {
            return false;
        } else if (pair_coder) {                     // give the two-per-compute-unit form up and start over
            pair_coder = false;
            i = 0;
        } else {
            return false;
        }
    }

    // ---- chunks ----
    out->pair_ok = out->pair_ok && pair_coder;
    if (!out->pair_ok && !plan_all(kTreeletWholeBuf, &all))
        return false;
    out->cost = cost_of(all);
    if (out->cost > limits.cost)
        return false;
    size_t largest = 0;
    out->max_trees = 0;
    out->chunks.clear();
    {
        size_t image_bytes = 0, n_ids = 0;
        int steps, entries, values;
        for (const std::vector<int> &b : all)
            for (size_t c = 0; c + 1 < b.size(); ++c) {
                image_bytes += chunk_size(b[c], b[c + 1], &steps, &entries, &values);
                n_ids += (size_t)values;
            }
        out->image.assign(image_bytes, 0);
        out->ids.assign(n_ids, 0);
    }
    size_t image_at = 0, ids_at = 0;
    struct Item { int32_t node, entry, step; };
    std::vector<Item> work;
    for (size_t si = 0; si < out->segments.size(); ++si) {
      TreeletSegmentPlan &sp = out->segments[si];
      sp.first_chunk = (int)out->chunks.size();
      sp.n_chunks = (int)all[si].size() - 1;
      for (size_t ci = 0; ci + 1 < all[si].size(); ++ci) {
        const int a = all[si][ci], b = all[si][ci + 1];
        TreeletChunk h;
        int steps, entries, values;
        const size_t bytes = chunk_size(a, b, &steps, &entries, &values);
        const int n = (b - a + kTreeletUnit - 1) / kTreeletUnit * kTreeletUnit;
        h.byte_off = (uint32_t)image_at;
        h.bytes = (uint32_t)bytes;
        h.n_trees = (uint32_t)n;
        h.first_tree = (uint32_t)a;
        h.n_real = (uint32_t)(b - a);
        h.val_off = (uint32_t)entries * 8u;
        h.steps = (uint32_t)steps;
        h.id_off = (uint32_t)ids_at;
        image_at += bytes;
        ids_at += (size_t)values;
        uint32_t *ent = (uint32_t *)(out->image.data() + h.byte_off);
        uint32_t *valtab = ent + 2 * (size_t)entries;
        uint16_t *ids = out->ids.data() + h.id_off;
        auto forced = [](int bit) -> uint32_t { return bit ? 0u : 255u; };
        auto absorb = [&](int32_t e) {               // an entry that steps onto itself
            const uint32_t t0 = forced((e >> 1) & 1), t1 = forced(e & 1);
            ent[2 * e] = t0 | ((uint32_t)(e >> 2) << 16);
            ent[2 * e + 1] = t1 | (t1 << 16);
        };
        int32_t next_entry = n, next_value = entries;
        for (int j = 0; j < n; ++j) {
            if (a + j >= b) {                        // padding
                absorb(j);
                const float minus_zero = -0.0f;
                memcpy(&valtab[j], &minus_zero, 4);
                continue;
            }
            const int32_t o = tree_off[a + j];
            work.clear();
            work.push_back({0, j, 0});
            for (size_t i = 0; i < work.size(); ++i) {
                const Item it = work[i];
                const int64_t g = (int64_t)o + it.node;
                if (sf[g] < 0) {
                    absorb(it.entry);
                    memcpy(&valtab[it.entry], &val[g], 4);
                    ids[it.entry] = (uint16_t)it.node;
                    continue;
                }
                const bool last = it.step + 1 == steps;
                int32_t &next = last ? next_value : next_entry;
                const int32_t block = next;
                next += 4;
                uint32_t half[2];
                const int32_t child[2] = {right[g], left[g]};
                for (int c = 0; c < 2; ++c) {
                    const int64_t gc = (int64_t)o + child[c];
                    int32_t to[2];                   // node of outcome (c, 0) and (c, 1), -1: never reached
                    if (sf[gc] < 0) {
                        half[c] = forced(1);
                        to[0] = -1;
                        to[1] = child[c];
                    } else {
                        half[c] = word[(size_t)gc];
                        to[0] = right[gc];
                        to[1] = left[gc];
                    }
                    for (int k = 0; k < 2; ++k) {
                        if (to[k] < 0)
                            continue;
                        const int32_t at = block + 2 * c + k;
                        if (last) {                  // the chunk's steps reach every leaf
                            memcpy(&valtab[at], &val[(int64_t)o + to[k]], 4);
                            ids[at] = (uint16_t)to[k];
                        } else {
                            work.push_back({to[k], at, it.step + 1});
                        }
                    }
                }
                ent[2 * it.entry] = word[(size_t)g] | ((uint32_t)(block >> 2) << 16);
                ent[2 * it.entry + 1] = half[0] | (half[1] << 16);
            }
        }
        largest = std::max(largest, bytes);
        out->max_trees = std::max(out->max_trees, n);
        out->chunks.push_back(h);
      }
    }
    out->buf_bytes = (int)largest;
    estimate_rounds(n_features, out);
    return true;
}

}  // namespace fs
