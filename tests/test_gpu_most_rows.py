"""Calls at the last row and program numbers that 32 bits hold."""
import numpy as np
import pytest

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


def test_as_many_programs_as_there_are_numbers(api):
    """All of them empty."""
    import torch
    off = torch.zeros(MOST + 1, dtype=torch.int32, device="cuda")
    score = torch.ones(MOST, device="cuda")
    api.fs_score_families([api.Family(model_without_trees(api, 0.5), None, api.FS_COLBLOCK64, 0, off, score)])
    assert not bool(score.any())
