"""Calls at the last row and program numbers that 32 bits hold."""
import numpy as np
import pytest

from paper_2201_00194_amd import workloads as W

pytestmark = pytest.mark.gpu
MOST = (1 << 31) - 1


@pytest.fixture(scope="module")
def api():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2201_00194_amd import api as A
    yield A
    torch.cuda.empty_cache()


def model_without_trees(api, bias):
    none = np.zeros(0, np.int32)
    return api.fs_model(1, np.zeros(1, np.int32), none, none.astype(np.float32), none, none, none.astype(np.float32), bias=bias)


@pytest.mark.parametrize("last", [100, 33])
def test_programs_that_end_at_the_last_row(api, last):
    """Long programs, then 64 whose rows are taken in windows that end there.  Every row's output is the bias: a row that is
    added twice or not at all shows."""
    import torch
    long_rows = MOST - 64 * last
    off = np.concatenate((np.linspace(0, long_rows, 65_537).astype(np.int64), long_rows + last * np.arange(1, 65))).astype(np.int32)
    score = torch.zeros(off.shape[0] - 1, device="cuda")
    x, outputs = torch.empty(api.fs_colblock64_floats(MOST, 1), device="cuda"), torch.empty(MOST, device="cuda")
    api.fs_score_families([api.Family(model_without_trees(api, 0.1), x, api.FS_COLBLOCK64, MOST, torch.from_numpy(off).cuda(), score,
                                      outputs)])
    lengths = np.diff(off)
    sums = np.add.accumulate(np.full(lengths.max(), 0.1, np.float32))          # one after the other
    assert np.array_equal(score.cpu().numpy().view(np.uint32), sums[lengths - 1].view(np.uint32))


@pytest.mark.parametrize("walk,rows", [("global", MOST), ("lds", MOST), ("treelet", MOST - 255), ("rank", MOST - 300), ("rank", MOST)])
def test_walks_end_at_the_last_row(api, oracle, tune, walk, rows):
    """As many rows as the walk takes (a launch has up to 2^32 - 1 threads, the rank walk makes two of what needs more).  All
    rows but the last few are zeros."""
    import torch
    tune(api.FS_TUNE_TREELET, 1 if walk == "treelet" else 0)
    tune(api.FS_TUNE_TREELET_FORM, 0)
    tune(api.FS_TUNE_RANK, 1 if walk == "rank" else 0)
    tune(api.FS_TUNE_RANK_TILES, 8)
    m = W.make_small_family(seed=11, n_programs=300, stmts=(1, 1), n_trees=4, depth=2, k=1, n_features=1, bias=0.25).model
    if walk == "global":
        m = W.Model(n_features=1, tree_off=np.zeros(1, np.int32), split_feature=m.split_feature[:0], threshold=m.threshold[:0],
                    left=m.left[:0], right=m.right[:0], value=m.value[:0], bias=0.25)
    last = 1000
    tail = np.random.default_rng(4).random((last, 1), np.float32)
    zero, expected = (oracle.score_programs(m, x, np.arange(x.shape[0] + 1, dtype=np.int32)) for x in (np.zeros((1, 1), np.float32), tail))
    x = torch.zeros(api.fs_colblock64_floats(MOST, 1), device="cuda")
    x[rows - last:rows] = torch.from_numpy(tail[:, 0]).cuda()
    off = torch.from_numpy(np.linspace(0, rows, 65_537).astype(np.int64).astype(np.int32)).cuda()
    score, outputs = torch.zeros(65_536, device="cuda"), torch.full((MOST + 640,), 7.0, device="cuda")
    model = api.fs_model.from_arrays(m)
    api.fs_score_families([api.Family(model, x, api.FS_COLBLOCK64, rows, off, score, outputs)])
    assert bool((outputs[:rows - last] == float(zero[0])).all())
    assert bool((outputs[rows:] == 7.0).all())                                # none is written past the last
    assert np.array_equal(outputs[rows - last:rows].cpu().numpy().view(np.uint32), expected.view(np.uint32))
    torch.cuda.synchronize()


def test_as_many_programs_as_there_are_numbers(api):
    """All of them empty."""
    import torch
    off = torch.zeros(MOST + 1, dtype=torch.int32, device="cuda")
    score = torch.ones(MOST, device="cuda")
    api.fs_score_families([api.Family(model_without_trees(api, 0.5), None, api.FS_COLBLOCK64, 0, off, score)])
    assert not bool(score.any())
