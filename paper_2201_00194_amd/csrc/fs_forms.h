// Host-side estimates of a scoring call's time, by which a call chooses between the two walks of a model
// that is prepared for both: byte-rank treelets and the LDS-staged format.
//
// Neither is the better one for a model.  Treelets pay for the coding of the rows (a latency that a short
// launch shows in full) and every walk of a chunk takes the steps of its deepest tree; the LDS walk pays
// for every level and for eight times the LDS reads.  Which one wins depends on layout and length of the call.
// Fitted to 597 models of 32 to 500 irregular or perfect trees of depth 4 to 12 on 24 to 250 features, 5 to
// 16 000 tiles, both layouts, with walks that were slower than they are now, the treelets' coder most of all.  Timed since,
// 80 models of 36 to 400 trees, depth 4 to 12 (perfect ones to 7), 1 to 8000 tiles, 1090 calls: the walk chosen takes 7.3 % more than
// the better one on the geometric mean, treelets alone 5.0 %, the LDS walk alone 32 %; 177 calls lose more than 10 %.
// (6.9 %, 5.9 % and 30 % with the coder before.)  Most of that are models of few trees with row-major or long calls, up to three
// times as long, which have no treelets at all because of the limit on their cost in fs_model_create.
#ifndef FS_FORMS_H
#define FS_FORMS_H

#include <math.h>

#include "fs_internal.h"

namespace fs {

// Row-major input needs no pass of its own where the first kernel to touch the features can
// read it: the rank-coding and treelet kernels always can; the LDS kernel transposes tiles on their way
// into LDS (through the still unused chunk region) when rows are whole 16-byte pieces and at
// least 8 padded rows fit below the tiles.  Other row-major families are re-tiled into scratch.
inline bool lds_reads_rowmajor(const fs_model *m)
{
    return m->n_features % 4 == 0 && m->lds_tile0 >= 8 * (m->n_features + 1) * 4;
}

// Form of the treelet kernel for a launch of so many tiles: long launches take two 4-tile workgroups per
// compute unit; when that leaves compute units idle, fewer tiles per workgroup whose wavefronts share the trees.
inline int treelet_form(int64_t tiles, int n_compute_units)
{
    if (tiles <= n_compute_units)
        return kTreeletSpread1;
    if (tiles <= 2 * n_compute_units)
        return kTreeletSpread2;
    if (tiles <= 4 * n_compute_units)
        return kTreeletSpread4;
    return kTreeletPair;
}

// Times the workgroups of a launch follow one another on a compute unit, one at a time: they keep in step for
// some rounds, then they spread.
inline double launch_rounds(double workgroups, int n_compute_units)
{
    const double r = workgroups / n_compute_units;
    return r <= 10.0 ? ceil(r) : r + 0.5;
}

// The same for two at a time.  One alone is the quicker: a last round of up to half the workgroups takes about
// 0.6 of a full one.
inline double launch_rounds_of_two(double workgroups, int n_compute_units)
{
    const double r = workgroups / (2.0 * n_compute_units), whole = floor(r);
    if (r > 3.0)
        return r + 0.5;
    return whole > 0.0 && r > whole && r <= whole + 0.5 ? whole + 0.6 : ceil(r);
}

// us of a call whose workgroups take `round_us` each (fs_model::tl_us, averaged over the families, as `once_us`:
// fs_model::tl_once_us).
inline double treelet_call_us(int form, double round_us, double once_us, double workgroups, int n_compute_units)
{
    if (form != kTreeletPair)
        return round_us;                             // such launches fit the chip
    return 11.0 + once_us + round_us * launch_rounds_of_two(workgroups, n_compute_units);
}

// Fetches of a tile group in the LDS walk: one per tile; row-major a part of a tile's rows at a time, as many as
// the kernel's staging area below the tiles takes.
inline double lds_fetches(const fs_model *m, bool rowmajor)
{
    const int rows = rowmajor ? m->lds_tile0 / (4 * (m->n_features + 1)) : 64;
    return m->lds_tiles * ceil(64.0 / (rows < 64 ? rows : 64));
}

// The same for the LDS walk: `group_us` = fs_model::lds_group_us, `fetches` as above, `group_features` = tiles x
// features of a group, all averaged; `form` is what the treelets would take, as a measure of the launch's length.
inline double lds_call_us(int form, bool rowmajor, double group_us, double fetches,
                          double group_features, double groups, int n_compute_units)
{
    struct Term { double call, fetch, feature; };
    static const Term terms[2][kTreeletForms] = {
        {{8.3, 0.2, 0.0079}, {5.7, 0.58, 0.0066}, {7.8, 0.0, 0.0029}, {7.2, 0.0, 0.0025}},
        {{7.0, 1.46, 0.0109}, {6.2, 1.58, 0.01}, {6.8, 1.4, 0.0079}, {5.8, 1.46, 0.0079}}};
    const Term &t = terms[rowmajor][form];
    return t.call + launch_rounds(groups, n_compute_units) *
                        (0.84 * group_us + t.fetch * fetches + t.feature * group_features);
}

// Rows of an odd number of features are re-tiled before the LDS walk reads them: a launch, latency up to some
// hundred tiles, then a rate.
inline double retile_us(double tile_features)
{
    return fmin(5.0 + 2.4e-4 * tile_features, 20.0 + 6e-5 * tile_features);
}

}  // namespace fs
#endif
