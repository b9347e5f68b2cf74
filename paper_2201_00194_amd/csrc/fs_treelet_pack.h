// Host-side result of packing a model into the byte-rank treelet format.
#ifndef FS_TREELET_PACK_H
#define FS_TREELET_PACK_H

#include <vector>

#include "fs_treelet.h"

namespace fs {

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
};

// False if the model does not fit the format (more columns than a byte names, a node graph that
// is not a tree, trees too large for a chunk -- or, unless `any_size`, so large that the other forms are
// as good; or with `pair_only`, where no two workgroups fit a compute unit).
bool build_treelets(int n_features, int n_trees, const int32_t *tree_off, const int32_t *sf,
                    const float *thr, const int32_t *left, const int32_t *right, const float *val,
                    bool any_size, bool pair_only, TreeletPlan *out);

}  // namespace fs
#endif
