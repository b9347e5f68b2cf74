"""Memory of training: what the calls allocate and wait for, batches trained in parts, and what is given back."""
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


def free_bytes():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def free_now():
    import torch
    return torch.cuda.mem_get_info()[0]


def sets_of(n, n_programs=400, n_features=164, max_cuts=20):
    return [W.make_train_set(60 + i, n_programs + 37 * i, stmts=(1, 6), n_features=n_features, max_cuts=max_cuts)
            for i in range(n)]


def test_boosting_neither_allocates_nor_waits(api):
    """Six trainers of depth 10 need more histograms than are kept between jobs; fs_trainer_create makes room for
    them, so that fs_train_boost only enqueues."""
    import torch
    sets = sets_of(6)
    params = api.train_params(max_depth=10, eta=0.5, lam=1.0)
    warm = api.fs_trainer.from_train_set(W.make_train_set(1, 50, n_features=5, max_cuts=3), max_depth=2, max_trees=1)
    api.fs_train_boost([warm], 1, api.train_params(max_depth=2, eta=0.5, lam=1.0))   # kernels and descriptors are there
    trs = [api.fs_trainer.from_train_set(ts, max_depth=10, max_trees=3) for ts in sets]
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    b = torch.mm(a, a)
    side = torch.cuda.Stream()
    before = free_bytes()
    busy = torch.cuda.Event()
    for _ in range(200):                             # 0.1 s of work on the default stream
        torch.mm(a, a, out=b)
    busy.record()
    api.fs_train_boost(trs, 2, params, stream=side)
    waited = busy.query()
    assert not waited, "fs_train_boost waited for another stream"
    torch.cuda.synchronize()
    assert before - free_bytes() < 16 << 20


def test_a_batch_in_parts_trains_like_one(api, T, tune):
    """Histograms of three trainers at a time at most: eight are trained in four parts, in two calls."""
    sets = sets_of(8, 300, 33)
    params = api.train_params(max_depth=6, eta=0.4, lam=1.0)
    tune(api.FS_TUNE_TRAIN_WORK_MB, 7)
    trs = [api.fs_trainer.from_train_set(ts, max_depth=6, max_trees=4) for ts in sets]
    api.fs_train_boost(trs, 2, params)
    api.fs_train_boost(trs[::-1], 1, params)
    for ts, tr in zip(sets, trs):
        exp = T.train(ts.features, ts.prog_off, ts.target, ts.cut_off, ts.cuts, n_rounds=3, max_depth=6, eta=0.4,
                      lam=1.0)
        same_trees(tr.export(), exp)
        assert tr.size()[0] == 3


def test_an_override_may_need_more_than_was_reserved(api, T, tune):
    ts = sets_of(1, 2500, 17, 63)[0]
    tr = api.fs_trainer.from_train_set(ts, max_depth=5, max_trees=2)
    tune(api.FS_TUNE_TRAIN_SLAB_ROWS, 64)
    api.fs_train_boost([tr], 2, api.train_params(max_depth=5, eta=0.4, lam=1.0))
    exp = T.train(ts.features, ts.prog_off, ts.target, ts.cut_off, ts.cuts, n_rounds=2, max_depth=5, eta=0.4, lam=1.0)
    same_trees(tr.export(), exp)


def test_one_plane_of_histograms_where_the_packed_form_cannot_overflow(api):
    """Six small families of depth 10 on 164 features: 512 nodes x 164 x 256 bins of eight bytes each."""
    sets = sets_of(6)
    before = free_bytes()
    trs = [api.fs_trainer.from_train_set(ts, max_depth=10, max_trees=1) for ts in sets]
    assert before - free_bytes() < 1_400_000_000     # 1.03 GB and what the buffer's steps add; two planes: 2.06 GB
    del trs


@pytest.mark.parametrize("packed", [-1, 0])
@pytest.mark.parametrize("n", [65_535, 65_536])
def test_both_sides_of_the_second_plane_with_saturated_gradients(api, T, tune, n, packed):
    """65 535 rows of programs of one row: curvature sums take 16 bits, and gradients at the fixed point's limit
    add up to just less than the 47 that are left.  With one row more the curvature takes 17 and the wide form
    may have to step in (here it does).  packed = 0: the wide form, which a trainer was not made for."""
    ts = W.make_train_set(9, n, stmts=(1, 1), n_features=5, max_cuts=31)
    ts.target[:] = np.where(ts.features[:, 2] < 0.5, 1e9, np.where(ts.features[:, 0] < 0.3, -1e9, 9e8)).astype(np.float32)
    params = api.train_params(max_depth=3, eta=0.5, lam=1.0)
    tr = api.fs_trainer.from_train_set(ts, max_depth=3, max_trees=2)
    tune(api.FS_TUNE_TRAIN_PACKED, packed)
    api.fs_train_boost([tr], 2, params)
    exp = T.train(ts.features, ts.prog_off, ts.target, ts.cut_off, ts.cuts, n_rounds=2, max_depth=3, eta=0.5, lam=1.0,
                  grad_scale=params.grad_scale)
    same_trees(tr.export(), exp)


def test_what_is_kept_is_given_back_where_memory_runs_out(api):
    """After the last trainer up to 512 MB stay.  A trainer, a scratch reservation or a model that is refused for
    want of memory has first taken them."""
    ts = W.make_train_set(3, 300, stmts=(1, 4), n_features=164, max_cuts=15)

    def keep():
        tr = api.fs_trainer.from_train_set(ts, max_depth=10, max_trees=1)
        api.fs_train_boost([tr], 1, api.train_params(max_depth=10, eta=0.5, lam=1.0))
        free_bytes()
        tr.destroy()
        return free_bytes()

    def refused(call):
        with pytest.raises(api.FsError) as e:
            call()
        assert e.value.code == api.FS_ENOMEM

    huge = 1 << 45                                   # 32 TB
    refused(lambda: api.fs_workspace_reserve(huge, 0))           # (the scratch of before is gone now)
    for call in (lambda: api.fs_trainer.from_train_set(ts, max_depth=10, max_trees=1 << 30),
                 lambda: api.fs_workspace_reserve(huge, 0)):
        kept = keep()
        refused(call)
        assert free_bytes() - kept > 150 << 20
    # a trainer alive keeps its buffer
    tr = api.fs_trainer.from_train_set(ts, max_depth=10, max_trees=2)
    alive = free_bytes()
    refused(lambda: api.fs_workspace_reserve(huge, 0))
    assert free_bytes() - alive < 16 << 20
    api.fs_train_boost([tr], 2, api.train_params(max_depth=10, eta=0.5, lam=1.0))
    assert tr.size()[0] == 2


@pytest.mark.parametrize("n_programs,n_features,max_cuts,depth,rounds", [
    (40, 5, 15, 3, 2),
    (300, 700, 255, 2, 2),                           # 0.7 MB of cut lists: more than is staged at once
    (6000, 17, 63, 10, 20),                          # 0.6 MB of trees
])
def test_a_destroyed_trainers_memory_serves_the_next(api, T, n_programs, n_features, max_cuts, depth, rounds):
    params = api.train_params(max_depth=depth, eta=0.4, lam=0.1)
    held = None
    for n in (n_programs, n_programs * 9 // 10):
        ts = W.make_train_set(n, n, stmts=(1, 6), n_features=n_features, max_cuts=max_cuts)
        tr = api.fs_trainer.from_train_set(ts, max_depth=depth, max_trees=rounds)
        api.fs_train_boost([tr], rounds, params)
        exp = T.train(ts.features, ts.prog_off, ts.target, ts.cut_off, ts.cuts, n_rounds=rounds, max_depth=depth,
                      eta=0.4, lam=0.1)
        same_trees(tr.export(), exp)
        tr.destroy()
        held = held or free_bytes()
        assert held - free_bytes() < 1 << 20         # the second one took no more


def keep_busy(stream, seconds=0.1):
    """An event on `stream` behind about so much work."""
    import torch
    a = torch.ones(8192, 8192, device="cuda", dtype=torch.bfloat16)
    b = torch.mm(a, a)
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for _ in range(int(seconds * 2000)):
            torch.mm(a, a, out=b)
        busy = torch.cuda.Event()
        busy.record()
    return busy, (a, b)                              # (to be kept until the stream is done)


def stream_of_its_own():
    """A stream whose work the default stream's does not queue up behind (streams share hardware queues)."""
    import torch
    one = torch.ones(64, device="cuda")
    for _ in range(8):
        side = torch.cuda.Stream()
        busy, held = keep_busy(side, 0.05)
        one.add_(1)
        torch.cuda.current_stream().synchronize()
        free = not busy.query()
        torch.cuda.synchronize()
        if free:
            return side
    pytest.skip("every stream tried shares a hardware queue with the default stream")


def maker(api, ts, **kw):
    """Creates trainers from inputs that are on the device already."""
    import torch
    n = ts.features.shape[1]
    x = api.fs_pack_colblock64(torch.from_numpy(ts.features).cuda(), ts.n_rows, n)
    off, y = torch.from_numpy(ts.prog_off.astype(np.int32)).cuda(), torch.from_numpy(ts.target.astype(np.float32)).cuda()
    torch.cuda.synchronize()
    return lambda max_trees: api.fs_trainer(n, x, api.FS_COLBLOCK64, ts.n_rows, off, ts.n_programs, y, ts.cut_off,
                                            ts.cuts, max_trees=max_trees, **kw)


@pytest.mark.parametrize("memory", ["fresh", "kept"])
def test_creating_a_trainer_waits_for_no_other_stream(api, memory):
    import torch
    create = maker(api, sets_of(1, 300, 17)[0], max_depth=4)
    side = stream_of_its_own()
    params = api.train_params(max_depth=4, eta=0.5, lam=1.0)
    first, other = create(50_000), create(50_000)    # 31 MB each (both alive: the histograms' buffer is large enough)
    api.fs_train_boost([first, other], 2, params)
    exported = other.export()
    torch.cuda.synchronize()
    first.destroy()
    busy, held = keep_busy(side)
    here = free_now()
    again = create(50_000 if memory == "kept" else 100_000)
    waited = busy.query()
    assert not waited, "fs_trainer_create waited for another stream"
    assert (here - free_now() < 16 << 20) == (memory == "kept")
    api.fs_train_boost([again], 2, params)
    for a, b in zip(again.export(), exported):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
    torch.cuda.synchronize()


@pytest.mark.parametrize("call", ["boost", "predictions"])
def test_what_a_destroyed_trainer_had_queued_is_waited_for(api, T, call):
    """Destroyed with work queued on another stream, behind more that is still running; its memory goes to the next."""
    import torch
    params = api.train_params(max_depth=6, eta=0.4, lam=0.1)
    sets = sets_of(2, 500, 23, 63)
    create_next, create_first = (maker(api, ts, max_depth=6) for ts in sets)
    side = stream_of_its_own()
    first = create_first(12_000)                     # 30 MB
    api.fs_train_boost([first], 1, params)
    torch.cuda.synchronize()
    busy, held = keep_busy(side)
    here = free_now()
    if call == "boost":
        api.fs_train_boost([first], 19, params, stream=side)
    else:
        with torch.cuda.stream(side):
            rows, progs = first.predictions(stream=side)
    assert not busy.query()
    first.destroy()
    following = create_next(12_000)
    assert here - free_now() < 16 << 20
    api.fs_train_boost([following], 3, params)
    ts = sets[0]
    same_trees(following.export(), T.train(ts.features, ts.prog_off, ts.target, ts.cut_off, ts.cuts, n_rounds=3,
                                           max_depth=6, eta=0.4, lam=0.1))
    torch.cuda.synchronize()
    if call == "predictions":
        ts = sets[1]
        exp = T.train(ts.features, ts.prog_off, ts.target, ts.cut_off, ts.cuts, n_rounds=1, max_depth=6, eta=0.4, lam=0.1)
        assert np.array_equal(rows.cpu().numpy().view(np.uint32), exp.row_pred.view(np.uint32))
        assert np.array_equal(progs.cpu().numpy().view(np.uint32), exp.prog_pred.view(np.uint32))


@pytest.mark.parametrize("order", ["bins first", "trees first"])
def test_whatever_kept_memory_holds(api, T, order):
    """One trainer's memory is nearly all random bins, the other's nearly all trees, most of which are never
    written: each finds what the other left where it expects to have cleared or written."""
    bins = W.make_train_set(71, 9000, stmts=(1, 4), n_features=40, max_cuts=255)
    trees = W.make_train_set(72, 200, stmts=(1, 3), n_features=6, max_cuts=40)
    shapes = [(bins, 3, 2), (trees, 10, 70)]         # 3.3 and 3.1 MB
    if order == "trees first":
        shapes = [(trees, 10, 78), (bins, 3, 2)]     # 3.4 and 3.3 MB
    held = None
    for ts, depth, most in shapes + shapes:
        tr = api.fs_trainer.from_train_set(ts, max_depth=depth, max_trees=most)
        api.fs_train_boost([tr], 2, api.train_params(max_depth=depth, eta=0.5, lam=1.0))
        exp = T.train(ts.features, ts.prog_off, ts.target, ts.cut_off, ts.cuts, n_rounds=2, max_depth=depth, eta=0.5, lam=1.0)
        same_trees(tr.export(), exp)
        tr.destroy()
        held = held or free_bytes()
        assert held - free_bytes() < 1 << 20         # one trainer's memory serves them all
