"""Which walks fs_model_create prepares a model for.  The plan is made on the host and reported on stderr
(FS_TUNE_VERBOSE), so this needs no GPU: without one the call fails behind it, when it asks for the device."""
import numpy as np
import pytest

from paper_2201_00194_amd import api, workloads as W


def perfect_model(n_features, n_used, n_trees, depth, zeros=0.3, seed=0):
    """Perfect trees, breadth-first ids; splits on the first n_used features, thresholds distinct but for the
    zeros, `zeros` of them all."""
    rng = np.random.default_rng([seed, n_features, n_trees, depth])
    nodes, splits = (2 << depth) - 1, (1 << depth) - 1
    inner = np.tile(np.arange(nodes) < splits, n_trees)
    child = np.tile(np.where(np.arange(nodes) < splits, 2 * np.arange(nodes) + 1, -1), n_trees)
    n = inner.shape[0]
    split = np.where(inner, rng.permutation(n) % n_used, -1).astype(np.int32)
    threshold = np.where(inner & (rng.random(n) >= zeros), (1 + rng.permutation(n)) / n, 0).astype(np.float32)
    value = np.where(inner, 0, rng.normal(size=n) * 0.1).astype(np.float32)
    return W.Model(n_features=n_features, tree_off=(np.arange(n_trees + 1) * nodes).astype(np.int32),
                   split_feature=split, threshold=threshold, left=child.astype(np.int32),
                   right=np.where(inner, child + 1, -1).astype(np.int32), value=value, bias=0.0)


def plan_of(capfd, tune, model):
    tune(api.FS_TUNE_VERBOSE, 1)
    capfd.readouterr()
    try:
        api.fs_model.from_arrays(model)
    except api.FsError as e:
        assert e.code == api.FS_EDEVICE
    return capfd.readouterr().err


@pytest.mark.parametrize("n_features,n_used,n_trees,treelets", [
    (164, 164, 300, True),         # two segments of 164 columns
    (164, 164, 500, False),        # three
    (200, 200, 200, True),         # one segment of 200
    (200, 200, 300, False),        # two
    (300, 180, 400, True),         # no LDS-staged form: two segments of 180 columns
    (300, 180, 540, False),        # three: the rank walk takes 511 features
])
def test_perfect_trees_of_depth_8_are_ranked_once_where_segments_would_code_them_often(capfd, tune, n_features, n_used,
                                                                                       n_trees, treelets):
    plan = plan_of(capfd, tune, perfect_model(n_features, n_used, n_trees, 8))
    assert ("treelets" in plan) == treelets
    assert ("rank-coded" in plan) == (not treelets)


def test_treelets_take_what_ranks_of_16_bits_cannot(capfd, tune):
    """17 425 thresholds of a feature are more than the rank walk's tables hold: then the many columns do not
    send the model to the walk from global memory."""
    plan = plan_of(capfd, tune, perfect_model(300, 6, 410, 8, zeros=0.0))
    assert "treelets" in plan and "rank-coded" not in plan


@pytest.mark.parametrize("n_features,n_trees,depth,early_leaf,both", [
    (230, 45, 12, 0.35, True),     # short calls belong to the LDS walk, long ones to treelets
    (164, 64, 7, 0.0, True),       # an odd depth: the last treelet step takes two levels for one
    (164, 200, 8, 0.2, True),
    (131, 100, 4, 0.0, True),
    (164, 300, 8, 0.0, False),     # the rank walk's, but for treelets
])
def test_a_model_has_both_walks_where_calls_differ(capfd, tune, n_features, n_trees, depth, early_leaf, both):
    if early_leaf == 0.0:
        model = perfect_model(n_features, n_features, n_trees, depth)
    else:
        rng = np.random.default_rng([n_features, n_trees])
        model = W.draw_model(rng, rng.random((4000, n_features), dtype=np.float32), n_trees, depth,
                             early_leaf_q=early_leaf)
    plan = plan_of(capfd, tune, model)
    assert "treelets" in plan
    assert ("trees per chunk:" in plan) == both
    assert "rank-coded" not in plan
