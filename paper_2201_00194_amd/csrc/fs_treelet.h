// Byte-rank treelet format: what fs_treelet.hip walks and fs_treelet_pack.hip builds.
//
// A split "x[f] < thr" only asks how x[f] orders against the thresholds the model itself uses on
// feature f.  With a feature's distinct thresholds sorted downwards, rank(x) = number of them > x and
// rank(thr) = 1 + position of thr,  x < thr  <=>  rank(x) >= rank(thr)  exactly; a NaN is below nothing,
// as it has rank 0 (counted upwards it would need a test of its own).  Up to
// kTreeletMaxCuts thresholds a rank fits a byte; a feature with more is split into several
// columns, each with its own piece of the sorted thresholds (x is below threshold p of a piece iff
// its rank inside that piece is above p, whatever the other pieces say).  Features the model
// does not use have no column.
//
// Columns in LDS: column c of four 64-row tiles is the 256 bytes at c*256, row l of tile t in byte
// 4*l + t: lane l reads bank l whichever column it asks for, and the address of a lane's value is
// (column << 8) | (4*lane + tile), one v_and_or of the node word.
//
// A treelet entry is 8 bytes {w0, w1}: a split node and its two children.
//     w0 = threshold rank (bits 0-7) | column (8-15) | block of the four outcomes (16-31)
//     w1 = right child: rank (0-7), column (8-15); left child: rank (16-23), column (24-31)
// A row goes left where its rank >= the threshold's; with b0, b1 the two decisions (1 = left) the walk goes
// on at entry 4*block + 2*b0 + b1 of the chunk.  Every walk of a chunk takes the chunk's `steps`
// steps (two levels each); what the last one yields indexes the chunk's value table.  A leaf above
// that level is an entry that steps onto itself: rank 0 (always left) or 255 (never: ranks stay
// below) force both decisions to its own position in its block, and the value table holds its
// value at its entry index.  Where a treelet's child is a leaf its own decision is forced too.
//
// A chunk image is [entries][values]: entries 0..n-1 are the roots of its trees, then the blocks;
// the value table covers the entry indices and, behind them, the outcomes of the last step.
// A chunk has a multiple of four trees; the last ones of a model may be padding (a single leaf
// with value -0, which no sum notices).
#ifndef FS_TREELET_H
#define FS_TREELET_H

#include <stdint.h>

namespace fs {

constexpr int kTreeletMaxCuts = 254;          // ranks 0..254; 255 is above every rank
constexpr int kTreeletMaxCols = 255;
constexpr int kTreeletLds = 80 * 1024;        // two workgroups per compute unit
constexpr int kTreeletLdsWhole = 160 * 1024;
// The coder moves the tables of a batch, up to 16 columns, in whole KB: what it reads behind the last column's.
// Twelve such batches have to fit the LDS of a compute unit, or the coder takes narrower ones.
constexpr int kTreeletTablePad = 16384;
constexpr int kTreeletMaxSegments = 16;
// Estimated clocks of a compute unit, per 64-row tile: coding a column, a step (two levels) of a tree,
// a chunk's barriers.
constexpr double kTreeletColClk = 18.0, kTreeletStepClk = 11.0, kTreeletChunkClk = 60.0;
constexpr int kTreeletFewTrees = 12;          // a chunk should hold at least about this many
constexpr int kTreeletMostRankCols = 399;     // of all segments, where the model could be rank-coded instead
constexpr int kTreeletMinTrees = 32;          // the coder's work needs trees to pay
constexpr int kTreeletUnit = 4;               // trees of a chunk come in units of four
// Trees of a chunk at most: two wavefronts of two rounds of twelve walks.  Chunks of the first kind
// fit one buffer beside the columns in half a compute unit's LDS; models with larger trees have chunks of
// the second kind and run one workgroup per compute unit.  (56 KB for models of few columns: -1 to +2 %.)
constexpr int kTreeletRound = 12;             // walks of a wavefront side by side
constexpr int kTreeletMaxTrees = 4 * kTreeletRound;
constexpr int kTreeletPairBuf = 40 * 1024;
constexpr int kTreeletSumBytes = 2048;
constexpr int kTreeletWholeBuf = 48 * 1024;
static_assert(kTreeletLdsWhole / 12 + 1024 <= kTreeletTablePad, "a batch of tables that starts at the last column");
static_assert(kTreeletLdsWhole - kTreeletMaxCols * 256 >= kTreeletWholeBuf + kTreeletMaxTrees * 1024,
              "a chunk and its value rows fit beside the widest columns");

struct TreeletChunk {
    uint32_t byte_off;      // into the image
    uint32_t bytes;         // multiple of 1024
    uint32_t n_trees;       // multiple of kTreeletUnit, padding included
    uint32_t first_tree;    // model-wide index of its first tree
    uint32_t n_real;        // trees that are not padding
    uint32_t val_off;       // byte offset of the value table in the chunk image
    uint32_t steps;         // >= 1
    uint32_t id_off;        // into the id map: caller's node id of value index v at [id_off + v]
};

// A column and how its ranks are found.  bucket(x) = x * scale + offset (one fused multiply-add, scale below 0) clamped
// to [0, 1], NaN to 0, times the number of buckets less one, rounded to the nearest integer: it never increases with x.
// The column's table gives for every bucket the number of thresholds in lower buckets (all > x) and `steps` bisection
// steps count those of x's own bucket (2^steps - 1 of them at most; thresholds of higher buckets are not above x, so a
// probe past the bucket's end counts nothing).  Table: `buckets` bytes, then the thresholds downwards, NaN behind.
struct TreeletCol {
    int32_t feature;
    float scale, offset;
    int32_t steps;
};

// Consecutive trees that share a set of columns.  An ensemble with more thresholds than 255 columns of
// 254 take is cut into segments; a workgroup codes its rows anew for each.
struct TreeletSegment {
    const TreeletCol *cols;
    const uint8_t *tables;        // [cols][table_stride], padded by kTreeletTablePad bytes
    int32_t n_cols;
    int32_t buckets;              // of every column, a multiple of 4
    int32_t table_stride;         // bytes, a multiple of 4
    int32_t first_chunk, n_chunks;
    int32_t pad;
};

// The device-resident description of a model in this format.
struct TreeletModel {
    const uint8_t *image;
    const TreeletChunk *chunks;
    const TreeletSegment *segments;
    const uint16_t *ids;
    int32_t n_segments;
    int32_t most_cols;            // of a segment: the chunks lie behind them
    int32_t buf_bytes;            // LDS a chunk takes at most, multiple of 1024
    int32_t max_trees;            // trees of the largest chunk
};

}  // namespace fs
#endif
