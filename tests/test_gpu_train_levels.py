"""Training from the smaller child of every split, against the training oracle, at the sizes where the
level's kernels change what they do: a node's rows just below, at and above one workgroup's share,
partition workgroups that are full or hold one row, feature groups of sixteen that are full or hold
one, families without a split, and batches whose families differ in all of this."""
import numpy as np
import pytest

from paper_2201_00194_amd import workloads as W
from test_gpu_train import check, same_trees

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2201_00194_amd import api as A
    return A


@pytest.fixture(scope="module")
def T():
    from oracle import train_oracle
    train_oracle.build()
    return train_oracle


def rows_set(seed, n, n_features, max_cuts=255):
    """n programs of one statement: exactly n rows."""
    return W.make_train_set(seed, n, stmts=(1, 1), n_features=n_features, max_cuts=max_cuts)


@pytest.mark.parametrize("packed", [-1, 0])
@pytest.mark.parametrize("n,n_features", [(1, 1), (2, 15), (63, 16), (64, 17), (65, 31), (127, 32), (128, 33), (129, 48),
                                          (511, 8), (512, 16), (513, 17), (1025, 193)])
def test_edges_of_rows_and_feature_groups(api, T, tune, packed, n, n_features):
    tune(api.FS_TUNE_TRAIN_SLAB_ROWS, 64)            # nodes of several workgroups' shares at these sizes
    tune(api.FS_TUNE_TRAIN_PACKED, packed)
    check(api, T, rows_set(n, n, n_features), rounds=2, max_depth=5, eta=0.5, lam=1.0)


@pytest.mark.parametrize("n", [65_536, 65_537])
def test_whole_moving_workgroups_and_a_row_more(api, T, n):
    """64 workgroups of 1024 rows move the root's records."""
    check(api, T, rows_set(7, n, 5, 31), rounds=2, max_depth=3, eta=0.5, lam=1.0)


@pytest.mark.parametrize("n,depth,rounds", [(12_288, 10, 2), (12_289, 2, 3), (49_152, 10, 1), (49_153, 10, 1), (49_153, 1, 3)])
def test_levels_grown_in_one_launch_and_moved_first(api, T, n, depth, rounds):
    """Both sides of the lines between the sizes of work items (12 288 rows) and between moving records in
    a launch of their own or with the histograms (49 152)."""
    check(api, T, rows_set(n, n, 5, 31), rounds=rounds, max_depth=depth, eta=0.5, lam=1.0)


@pytest.mark.parametrize("programs,slab,packed", [(900, 64, -1), (900, 64, 0), (9000, 128, -1), (9000, 128, 0)])
def test_counted_children_of_uneven_programs(api, T, tune, programs, slab, packed):
    """Programs of 1..12 rows: the child of less curvature may hold more rows; nodes of many pieces."""
    ts = W.make_train_set(programs, programs, stmts=(1, 12), n_features=19, max_cuts=63)
    assert (ts.n_rows > 49_152) == (programs == 9000)
    tune(api.FS_TUNE_TRAIN_SLAB_ROWS, slab)
    tune(api.FS_TUNE_TRAIN_PACKED, packed)
    check(api, T, ts, rounds=2, max_depth=7, eta=0.5, lam=1.0)


@pytest.mark.parametrize("programs,stmts", [(65, (15, 17)), (64, (16, 16)), (300, (1, 50)), (10_000, (1, 3)), (10_001, (1, 3))])
def test_gradients_of_long_programs_and_of_many(api, T, programs, stmts):
    """Around the sixteen rows of a program that are held for its records, and on both sides of the line between
    workgroups of one wavefront and of four."""
    ts = W.make_train_set(programs + stmts[1], programs, stmts=stmts, n_features=5, max_cuts=31)
    check(api, T, ts, rounds=3, max_depth=3, eta=0.5, lam=1.0)


def test_second_boost_goes_deeper_and_a_family_without_a_split(api, T):
    import torch
    sets = [rows_set(3, 3000, 20), rows_set(4, 1, 3), W.make_train_set(5, 700, stmts=(1, 9), n_features=164, max_cuts=63)]
    trs = [api.fs_trainer.from_train_set(s, max_depth=10, max_trees=4) for s in sets]
    p = [api.train_params(max_depth=k, eta=0.4, lam=0.0) for k in (1, 10)]
    api.fs_train_boost(trs, 1, p[0])
    api.fs_train_boost(trs[:1], 2, p[1])             # the histogram places of a deeper tree
    api.fs_train_boost(trs[1:], 2, p[1])
    torch.cuda.synchronize()
    for s, tr in zip(sets, trs):
        first = T.train(s.features, s.prog_off, s.target, s.cut_off, s.cuts, n_rounds=1, max_depth=1, eta=0.4, lam=0.0)
        got = tr.export()
        n = int(first.tree_off[1])
        assert int(got[0][1]) == n and np.array_equal(got[1][:n], first.split_feature)
        assert np.array_equal(got[5][:n].view(np.uint32), first.value.view(np.uint32))
        then = T.train(s.features, s.prog_off, s.target, s.cut_off, s.cuts, n_rounds=2, max_depth=10, eta=0.4, lam=0.0,
                       start=first.row_pred)
        later = [a[n:] for a in got[1:]]
        same_trees([got[0][1:] - n] + later, then)
        # and through the outputs they leave: the rows' walk of all trees, in their order
        to, sf, th, le, ri, va = got
        out = np.zeros(s.n_rows, np.float32)
        for t in range(len(to) - 1):
            at = np.zeros(s.n_rows, np.int64)
            for _ in range(11):
                g = to[t] + at
                inner = sf[g] >= 0
                x = s.features[np.arange(s.n_rows), np.maximum(sf[g], 0)]
                at = np.where(inner, np.where(x < th[g], le[g], ri[g]), at)
            out = out + va[to[t] + at]
        rows, _ = tr.predictions()
        torch.cuda.synchronize()
        assert np.array_equal(rows.cpu().numpy().view(np.uint32), out.view(np.uint32))
