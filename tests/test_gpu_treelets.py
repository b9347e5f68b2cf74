"""The byte-rank treelet traversal (fs_treelet.hip) against the oracle: every output of every form of
the kernel, at the edges of its format -- tiles and rounds that are not full, features with more
thresholds than one column holds, ensembles cut into segments, leaves at every depth, special
values, both layouts."""
import numpy as np
import pytest

from paper_2201_00194_amd import workloads as W
from test_gpu_parity import check_family, run_families

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2201_00194_amd import api as A
    return A


def family(seed, n_programs, stmts, n_trees, depth, q, n_features=164, special=False, steps=0):
    fam = W.make_small_family(seed=seed, n_programs=n_programs, stmts=stmts, n_trees=n_trees, depth=depth,
                              early_leaf_q=q, n_features=n_features, k=min(50, n_programs), bias=0.5)
    rng = np.random.default_rng(seed)
    if steps:                                   # few distinct values: thresholds and features tie
        fam.features[:] = np.floor(fam.features * steps) / steps
        fam.model.threshold[:] = np.where(fam.model.split_feature >= 0,
                                          np.floor(fam.model.threshold * steps) / steps, 0)
    if special:
        X = fam.features
        inner = np.flatnonzero(fam.model.split_feature >= 0)
        for val in (np.nan, np.inf, -np.inf, -0.0, 1e-42, -1e-42, 3e38, -3e38):
            X[rng.integers(0, X.shape[0], 60), rng.integers(0, X.shape[1], 60)] = val
            fam.model.threshold[rng.choice(inner, min(5, inner.size), replace=False)] = val
    return fam


CASES = [
    # one row; a tile and a row; four tiles and a row; trees that fill no unit, one unit, a round and one
    dict(n_programs=1, stmts=(1, 1), n_trees=33, depth=5, q=0.2),
    dict(n_programs=65, stmts=(1, 1), n_trees=4, depth=3, q=0.0),
    dict(n_programs=257, stmts=(1, 1), n_trees=49, depth=7, q=0.25, special=True),
    # single leaves, stumps, an odd depth; the narrowest and the widest feature matrix
    dict(n_programs=150, stmts=(1, 3), n_trees=35, depth=0, q=0.0),
    dict(n_programs=90, stmts=(2, 2), n_trees=97, depth=1, q=0.0, n_features=1, special=True),
    dict(n_programs=120, stmts=(1, 4), n_trees=60, depth=5, q=0.1, n_features=255),
    dict(n_programs=130, stmts=(1, 4), n_trees=70, depth=6, q=0.3, n_features=131, steps=3),
    # more thresholds per feature than a column holds; two segments; deep irregular trees
    dict(n_programs=300, stmts=(3, 5), n_trees=50, depth=8, q=0.0, n_features=30, special=True),
    dict(n_programs=500, stmts=(4, 8), n_trees=280, depth=8, q=0.0),
    dict(n_programs=200, stmts=(1, 9), n_trees=90, depth=12, q=0.3, special=True),
]


@pytest.mark.parametrize("form", [-1, 0, 1, 2, 3])
@pytest.mark.parametrize("layout", [0, 1])
def test_treelet_forms_all_outputs(api, oracle, tune, form, layout):
    tune(api.FS_TUNE_TREELET, 1)
    tune(api.FS_TUNE_TREELET_FORM, form)
    fams = [family(9000 + i, **c) for i, c in enumerate(CASES)]
    devs = run_families(api, fams, layout)
    for f, d in zip(fams, devs):
        check_family(oracle, f, d)
    devs = run_families(api, fams, layout, want_rows=False, want_leaves=False)
    for f, d in zip(fams, devs):
        check_family(oracle, f, d)


@pytest.mark.parametrize("seed", range(12))
def test_treelets_random_shapes(api, oracle, tune, seed):
    rng = np.random.default_rng([seed, 424])
    tune(api.FS_TUNE_TREELET, 1)
    tune(api.FS_TUNE_TREELET_FORM, int(rng.integers(-1, 4)))
    fams = []
    for i in range(4):
        depth = int(rng.integers(0, 11))
        fams.append(family(7000 + 10 * seed + i, int(rng.integers(1, 300)), (1, int(rng.integers(1, 12))),
                           int(rng.integers(1, 30 if depth > 8 else 120)), depth,
                           float(rng.choice([0.0, 0.15, 0.35])), n_features=int(rng.choice([2, 33, 64, 164, 255, 300])),
                           special=bool(rng.integers(0, 2)), steps=int(rng.choice([0, 0, 2, 40]))))
    devs = run_families(api, fams, int(rng.integers(0, 2)))
    for f, d in zip(fams, devs):
        check_family(oracle, f, d)


# A model with both walks, the layout, the rows of a call that belongs to the LDS walk and of one that
# belongs to treelets: the coding shows in short calls; row-major input takes the coder longer in long ones.
# 230 features row-major are re-tiled for the LDS walk, 24 and 164 are not.
CHOICES = [
    (dict(n_trees=100, depth=10, q=0.3, n_features=230), 1, 300, 150000),
    (dict(n_trees=32, depth=8, q=0.35, n_features=24), 1, 64, 400000),
    (dict(n_trees=160, depth=12, q=0.35, n_features=230), 0, 300, 40000),
    (dict(n_trees=100, depth=7, q=0.0, n_features=164), 0, 126000, None),
    (dict(n_trees=100, depth=6, q=0.2, n_features=164), 0, None, 257),
]


@pytest.mark.parametrize("shape,layout,lds_rows,treelet_rows", CHOICES)
def test_the_call_chooses_between_the_walks(api, oracle, tune, capfd, shape, layout, lds_rows, treelet_rows):
    tune(api.FS_TUNE_VERBOSE, 1)
    sizes = {}
    for rows, treelets in ((lds_rows, False), (treelet_rows, True)):
        if rows is None:
            continue
        fam = family(8100, 3000, (1, 1), special=True, **shape)
        if rows > 3000:
            fam.features = np.random.default_rng(3).random((rows, shape["n_features"]), dtype=np.float32)
            fam.prog_off = np.arange(0, rows + 1, 4, dtype=np.int32)
        else:
            fam.features, fam.prog_off = fam.features[:rows], fam.prog_off[:rows + 1]
        fam.k = 50
        capfd.readouterr()
        dev, = run_families(api, [fam], layout, want_rows=rows <= 100000, want_leaves=rows <= 50000)
        plan = capfd.readouterr().err
        assert "treelets," in plan                   # the model has them
        assert ("1 of 1 families walk treelets" in plan) == treelets and ("LDS shape" in plan) == (not treelets)
        check_family(oracle, fam, dev)
        sizes[rows] = api.fs_workspace_bytes([dev.family()])
    # scratch reserved for the long call serves the short one, whichever walk it takes
    assert sizes[min(sizes)] <= sizes[max(sizes)]


@pytest.mark.parametrize("layout", [0, 1])
def test_one_call_with_every_walk(api, oracle, layout):
    """Families whose models have both walks beside some that have one: 230 features (re-tiled where row-major),
    24 (not), perfect trees that stay treelets, ranked ones, more than 255 features by treelets and, with few trees,
    from global memory."""
    fams = [family(8200 + i, n, (1, 3), special=True, **c) for i, (n, c) in enumerate([
        (90, dict(n_trees=45, depth=12, q=0.35, n_features=230)),
        (70, dict(n_trees=32, depth=8, q=0.35, n_features=24)),
        (1, dict(n_trees=100, depth=12, q=0.35, n_features=230)),
        (120, dict(n_trees=60, depth=8, q=0.0, n_features=64)),
        (65, dict(n_trees=20, depth=9, q=0.0, n_features=64)),
        (40, dict(n_trees=5, depth=6, q=0.2, n_features=300)),
        (130, dict(n_trees=32, depth=4, q=0.0, n_features=300)),
        (33, dict(n_trees=20, depth=5, q=0.2, n_features=131))])]
    devs = run_families(api, fams, layout)
    for f, d in zip(fams, devs):
        check_family(oracle, f, d)


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("n_features,n_trees,depth,q", [(250, 60, 8, 0.2), (255, 48, 7, 0.1), (236, 45, 9, 0.25), (110, 300, 9, 0.2)])
def test_columns_that_leave_room_for_one_table_a_wavefront(api, oracle, tune, layout, n_features, n_trees, depth, q):
    """Many columns in half a compute unit's LDS: the coder's tables have no second buffer."""
    tune(api.FS_TUNE_TREELET, 1)
    tune(api.FS_TUNE_TREELET_FORM, 0)
    fam = family(n_features, 560, (2, 5), n_trees, depth, q, n_features=n_features, special=True)
    check_family(oracle, fam, run_families(api, [fam], layout)[0])


def test_a_large_model_with_both_walks(api, oracle):
    """112 000 nodes: the two formats are built side by side; calls on both sides of the choice."""
    fam = family(5, 200, (1, 2), 400, 12, 0.3)
    big = family(6, 3000, (16, 16), 150, 12, 0.3, n_features=200)
    for f, dev in zip([fam, big], run_families(api, [fam, big], 0, want_leaves=False)):
        check_family(oracle, f, dev, check_leaves=False)
    check_family(oracle, fam, run_families(api, [fam], 1)[0])
