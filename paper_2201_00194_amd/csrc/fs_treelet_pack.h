// Host-side result of packing a model into the byte-rank treelet format.
#ifndef FS_TREELET_PACK_H
#define FS_TREELET_PACK_H

#include <limits.h>
#include <math.h>
#include <algorithm>
#include <vector>

#include "fs_internal.h"
#include "fs_treelet.h"

namespace fs {

// Shapes of a model's trees, collected while its nodes are validated.
struct TreeShapes {
    static constexpr int kMaxSteps = 32;             // level pairs the treelet format is meant for
    struct Tree {
        int32_t n_split, n_leaf;                     // on the paths from the root
        int32_t depth;                               // splits to the deepest leaf
        bool tree;                                   // no node has two parents
        bool perfect;                                // all leaves at one depth, 1 to 14
    };
    std::vector<Tree> trees;
    // splits at depth 2*s of the trees before t, at [s][t] (empty: there are none)
    std::vector<int32_t> sum[kMaxSteps];
    bool deep = false;                               // some split lies deeper than that

    void begin_tree() { std::fill(here_, here_ + kMaxSteps, 0); }
    void add_split(int32_t level)
    {
        if (level >= 2 * kMaxSteps)
            deep = true;
        else if ((level & 1) == 0)
            ++here_[level / 2];
    }
    void end_tree(int t, int n_trees)
    {
        for (int s = 0; s < kMaxSteps; ++s) {
            if (sum[s].empty()) {
                if (here_[s] == 0)
                    break;                           // no splits at deeper levels either
                sum[s].assign((size_t)n_trees + 1, 0);
            }
            sum[s][(size_t)t + 1] = sum[s][(size_t)t] + here_[s];
        }
    }
    // treelet steps (two levels each) to tree t's deepest leaf, at least 1
    int steps(int t) const { return std::max(1, (trees[(size_t)t].depth + 1) / 2); }
    int max_depth() const
    {
        int d = 0;
        for (const Tree &t : trees)
            d = std::max(d, (int)t.depth);
        return d;
    }
    // the trees' depth if all are perfect and of one depth, else -1
    int perfect_depth() const
    {
        for (const Tree &t : trees)
            if (!t.perfect || t.depth != trees[0].depth)
                return -1;
        return trees.empty() ? -1 : (int)trees[0].depth;
    }

private:
    int32_t here_[kMaxSteps];
};

struct TreeletSegmentPlan {
    int first_tree = 0, n_trees = 0;
    std::vector<TreeletCol> cols;
    std::vector<uint8_t> tables;
    int buckets = 0, table_stride = 0, first_chunk = 0, n_chunks = 0;
};

struct TreeletPlan {
    std::vector<uint8_t> image;
    std::vector<TreeletChunk> chunks;
    std::vector<TreeletSegmentPlan> segments;
    std::vector<uint16_t> ids;
    int most_cols = 0, buf_bytes = 0, max_trees = 0;
    bool pair_ok = false;         // a chunk buffer fits beside the columns in half a compute unit's LDS
    double cost = 0.0;            // clocks of a compute unit per 64-row tile, estimated
    float us[2][kTreeletForms] = {};   // a round of a launch, estimated: fs_model::tl_us
    float once_us = 0.0f;              // fs_model::tl_once_us
};

// What a plan may not exceed, found out as early as possible.
struct TreeletLimits {
    bool any_size = true;         // also trees so large that the other forms are as good
    bool pair_only = false;       // only if two workgroups fit a compute unit
    double cost = HUGE_VAL;       // clocks, as TreeletPlan::cost
    int cols = INT_MAX;           // columns of all segments together
    bool ranks = false;           // the rank walk could take the model
};

// False if the model does not fit the format (more columns than a byte names, a node graph that
// is not a tree, trees too large for a chunk) or exceeds a limit.
bool build_treelets(int n_features, int n_trees, const TreeShapes &shape, const int32_t *tree_off,
                    const int32_t *sf, const float *thr, const int32_t *left, const int32_t *right, const float *val,
                    const TreeletLimits &limits, TreeletPlan *out);

}  // namespace fs
#endif
