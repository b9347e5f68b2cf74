"""The rank walk's slots: wavefronts that walk and replace their own trees and hand a row's sum on in tree order.
All tile counts, fewer trees than slots, last turns that are not full, a last workgroup with tiles missing, trees
larger than the registers they are prefetched into; every leaf and every bit against the oracle."""
import numpy as np
import pytest

from paper_2201_00194_amd import workloads as W
from test_gpu_parity import api, check_family, run_families  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [1, 2, 3, 4, 6])
@pytest.mark.parametrize("depth,trees,rows", [(3, 1, 1), (8, 2, 65), (8, 97, 64 * 13 + 5), (9, 25, 64 * 6), (10, 41, 64 * 7 + 1),
                                              (11, 7, 130), (12, 5, 64 * 4 - 1)])
def test_slots_at_their_edges(api, oracle, tune, tiles, depth, trees, rows):  # noqa: F811
    tune(api.FS_TUNE_RANK, 1)
    tune(api.FS_TUNE_RANK_TILES, tiles)
    fam = W.make_small_family(seed=1000 + depth + trees, n_programs=rows, stmts=(1, 1), n_trees=trees, depth=depth, k=5,
                              bias=0.25)
    devs = run_families(api, [fam], api.FS_COLBLOCK64)
    check_family(oracle, fam, devs[0])


@pytest.mark.parametrize("tiles", [5, 8])
@pytest.mark.parametrize("depth,trees,features", [(1, 33, 20), (2, 9, 20), (9, 150, 70), (10, 41, 33), (12, 11, 40)])
def test_more_tiles_than_four(api, oracle, tune, tiles, depth, trees, features):  # noqa: F811
    tune(api.FS_TUNE_RANK, 1)
    tune(api.FS_TUNE_RANK_TILES, tiles)
    fam = W.make_small_family(seed=depth + trees, n_programs=64 * 11 + 3, stmts=(1, 1), n_trees=trees, depth=depth, k=5,
                              n_features=features)
    check_family(oracle, fam, run_families(api, [fam], api.FS_COLBLOCK64)[0])


@pytest.mark.parametrize("tiles", [1, 7, 256, 257, 520, 900, 2100])
def test_workgroups_follow_the_length_of_the_call(api, oracle, tune, tiles):  # noqa: F811
    """So many tiles take one, two, three ... of them a workgroup; a family of a few rows beside them takes no more than it has."""
    tune(api.FS_TUNE_RANK, 1)
    fams = [W.make_small_family(seed=tiles, n_programs=64 * tiles - 5, stmts=(1, 1), n_trees=70, depth=8, k=5, n_features=24),
            W.make_small_family(seed=tiles + 1, n_programs=90, stmts=(1, 1), n_trees=17, depth=9, k=5, n_features=164)]
    for n in (1, 2):
        for f, dev in zip(fams[:n], run_families(api, fams[:n], api.FS_COLBLOCK64)):
            check_family(oracle, f, dev)


@pytest.mark.parametrize("depth,trees", [(10, 150), (11, 100), (12, 41)])
def test_more_registers_than_the_kernel_has(api, oracle, tune, depth, trees):  # noqa: F811
    """One tile a workgroup and several turns of 10, 12 and 16 registers a thread: what eight do not hold is read later."""
    tune(api.FS_TUNE_RANK, 1)
    tune(api.FS_TUNE_RANK_TILES, 1)
    features = 100 if depth == 12 else 164
    fam = W.make_small_family(seed=depth, n_programs=64 * 3 + 5, stmts=(1, 1), n_trees=trees, depth=depth, k=5, n_features=features)
    check_family(oracle, fam, run_families(api, [fam], api.FS_COLBLOCK64)[0])


def test_a_few_rows_do_not_decide_the_registers(api, oracle, tune, capfd):  # noqa: F811
    tune(api.FS_TUNE_RANK, 1)
    fams = [W.make_small_family(seed=5, n_programs=64 * 2000, stmts=(1, 1), n_trees=300, depth=7, k=5, n_features=30),
            W.make_small_family(seed=6, n_programs=60, stmts=(1, 1), n_trees=100, depth=11, k=5, n_features=164)]
    tune(api.FS_TUNE_VERBOSE, 1)
    said = []
    for some in (fams[:1], fams[1:], fams):
        capfd.readouterr()
        devs = run_families(api, some, api.FS_COLBLOCK64)
        said += [int(line.split()[-2]) for line in capfd.readouterr().err.splitlines() if "registers" in line]
        for f, dev in zip(some, devs):
            check_family(oracle, f, dev)
    alone, few, both = said
    assert few > 8 and both == alone < few


def test_models_of_different_trees_in_one_launch(api, oracle, tune):  # noqa: F811
    tune(api.FS_TUNE_RANK, 1)
    fams = [W.make_small_family(seed=70 + d, n_programs=90 + 31 * d, stmts=(1, 4), n_trees=3 + 11 * (12 - d), depth=d, k=8)
            for d in (12, 4, 8, 10)]
    for f, dev in zip(fams, run_families(api, fams, api.FS_COLBLOCK64)):
        check_family(oracle, f, dev)


@pytest.mark.parametrize("depth,features", [(8, 164), (8, 180), (8, 251), (9, 100), (9, 164), (2, 510), (1, 511), (2, 600), (0, 9)])
def test_last_splits_and_leaf_values_in_memory(api, oracle, tune, depth, features):  # noqa: F811
    """Whatever the depth and the room beside the tiles.  (More than 511 features and trees of one leaf take other walks.)"""
    tune(api.FS_TUNE_RANK, 1)
    fam = W.make_small_family(seed=depth + features, n_programs=64 * 9 + 7, stmts=(1, 1), n_trees=53, depth=depth, k=5,
                              n_features=features, bias=-0.5)
    check_family(oracle, fam, run_families(api, [fam], api.FS_COLBLOCK64)[0])


@pytest.mark.parametrize("kind", ["spread", "one value", "crowded", "decades", "with infinities"])
@pytest.mark.parametrize("layout", ["colblock", "rowmajor"])
def test_thresholds_in_buckets_or_search_trees(api, oracle, tune, kind, layout):  # noqa: F811
    """The coder's tables follow how a feature's thresholds are spread; values are on, beside and far off them."""
    tune(api.FS_TUNE_RANK, 1)
    fam = W.make_small_family(seed=31, n_programs=700, stmts=(1, 2), n_trees=40, depth=6, k=5, n_features=13)
    rng = np.random.default_rng(8)
    m, x = fam.model, fam.features
    split = np.flatnonzero(np.asarray(m.split_feature) >= 0)
    n = split.shape[0]
    thr = np.array(m.threshold, np.float32)
    if kind == "one value":
        thr[split] = 0.25
    elif kind == "crowded":
        thr[split] = np.where(rng.random(n) < 0.9, 1.0 + rng.integers(0, 200, n) * 2.0 ** -23, rng.random(n) * 1e6)
    elif kind == "decades":
        thr[split] = 10.0 ** rng.uniform(-38, 38, n) * rng.choice([-1, 1], n)
    elif kind == "with infinities":
        thr[split] = np.where(rng.random(n) < 0.1, rng.choice([np.inf, -np.inf, 0.0, -0.0, np.nan], n), rng.random(n))
    m.threshold[:] = thr
    pick = rng.random(x.shape)
    near = thr[split][rng.integers(0, n, x.shape)]
    x[:] = np.where(pick < 0.4, near, np.where(pick < 0.6, np.nextafter(near, np.float32(np.inf)),
                    np.where(pick < 0.7, rng.choice([np.inf, -np.inf, np.nan, 0.0, -0.0, 1e-45], x.shape), x)))
    check_family(oracle, fam, run_families(api, [fam], getattr(api, "FS_" + layout.upper() + ("64" if layout == "colblock" else "")))[0])


@pytest.mark.parametrize("crowd", [6, 7, 8, 14, 15, 16, 17, 40])
def test_buckets_of_as_many_thresholds_as_the_steps_find(api, oracle, tune, crowd):  # noqa: F811
    """So many thresholds of one feature lie closer together than buckets are wide, the others far apart: 2^steps - 1 of
    them are the most that buckets serve (15; beyond that the search tree)."""
    tune(api.FS_TUNE_RANK, 1)
    fam = W.make_small_family(seed=90 + crowd, n_programs=500, stmts=(1, 2), n_trees=6, depth=5, k=5, n_features=3)
    rng = np.random.default_rng(crowd)
    m, x = fam.model, fam.features
    thr = np.array(m.threshold, np.float32)
    for f in range(3):
        of = rng.permutation(np.flatnonzero(np.asarray(m.split_feature) == f))
        assert of.shape[0] > crowd + 5
        thr[of] = np.linspace(0, 1, of.shape[0])
        if f == 1:
            thr[of[:crowd]] = 0.503 + np.arange(crowd) * 1e-6
    m.threshold[:] = thr
    near = thr[rng.integers(0, thr.shape[0], x.shape)]
    x[:] = np.where(rng.random(x.shape) < 0.5, np.where(rng.random(x.shape) < 0.5, near, np.nextafter(near, np.float32(-1))),
                    0.503 + rng.integers(-3, 45, x.shape) * 1e-6)
    check_family(oracle, fam, run_families(api, [fam], api.FS_COLBLOCK64)[0])
