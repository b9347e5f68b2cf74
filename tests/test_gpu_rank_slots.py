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


def test_models_of_different_trees_in_one_launch(api, oracle, tune):  # noqa: F811
    tune(api.FS_TUNE_RANK, 1)
    fams = [W.make_small_family(seed=70 + d, n_programs=90 + 31 * d, stmts=(1, 4), n_trees=3 + 11 * (12 - d), depth=d, k=8)
            for d in (12, 4, 8, 10)]
    for f, dev in zip(fams, run_families(api, fams, api.FS_COLBLOCK64)):
        check_family(oracle, f, dev)


@pytest.mark.parametrize("depth,features", [(8, 164), (8, 180), (8, 251), (9, 100), (9, 164), (2, 600), (1, 630), (0, 9)])
def test_leaf_values_in_lds_or_in_memory(api, oracle, tune, depth, features):  # noqa: F811
    """They are held where that leaves room for 64 trees walked at a time on six tiles, and always in shallow trees."""
    tune(api.FS_TUNE_RANK, 1)
    fam = W.make_small_family(seed=depth + features, n_programs=64 * 9 + 7, stmts=(1, 1), n_trees=53, depth=depth, k=5,
                              n_features=features, bias=-0.5)
    check_family(oracle, fam, run_families(api, [fam], api.FS_COLBLOCK64)[0])
