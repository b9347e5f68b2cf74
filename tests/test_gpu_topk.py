"""Cuts at the sizes where their kernels change over, on scores with ties, zeros of both signs, infinities and NaN."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SCORES = {
    "random": lambda g, n: g.standard_normal(n),
    "equal": lambda g, n: np.full(n, -0.25),
    "few values": lambda g, n: g.integers(0, 5, n) / 4 - 0.5,
    "close": lambda g, n: 1.0 + g.integers(0, 3000, n) * 2.0 ** -23,          # the first pass of the select tells none apart
    "special": lambda g, n: g.choice([0.0, -0.0, np.inf, -np.inf, np.nan, 1e-45, -1e-45, 1.0], n),
}


@pytest.fixture(scope="module")
def api():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2201_00194_amd import api as A
    return A


@pytest.mark.parametrize("kind", SCORES)
@pytest.mark.parametrize("n,k", [(1, 1), (63, 64), (255, 255), (256, 16), (257, 1), (257, 256), (321, 320), (321, 321),
                                 (1025, 320), (1025, 456), (513, 512), (600, 513), (4096, 64), (8191, 321), (8192, 64), (9001, 2000), (200_000, 64), (1024, 1024), (1500, 1025),
                                 (2048, 2048), (3000, 2500), (4097, 4096), (8191, 8191), (8000, 4097), (20_000, 16_384),
                                 (1_100_000, 16_384), (8200, 5000), (18_000, 6000), (34_000, 5000), (262_200, 4097)])
def test_cut(api, oracle, kind, n, k):
    import torch
    score = SCORES[kind](np.random.default_rng([n, k]), n).astype(np.float32)
    d = torch.from_numpy(score).cuda()
    idx = torch.zeros(k, dtype=torch.int32, device="cuda")
    best = torch.zeros(k, dtype=torch.float32, device="cuda")
    api.fs_topk([api.TopkRequest(d, n, k, idx, best)])
    e_idx, e_best = oracle.topk(score, k)
    assert np.array_equal(idx.cpu().numpy(), e_idx)
    assert np.array_equal(best.cpu().numpy().view(np.uint32), e_best.view(np.uint32))


@pytest.mark.parametrize("kind", ["random", "equal", "special"])
@pytest.mark.parametrize("sizes", [[(8192, 256)], [(8193, 257)], [(16_383, 64), (9001, 50)], [(16_384, 256), (1, 1)], [(16_385, 64)],
                                   [(12_000, 64), (16_385, 64)], [(12_000, 64), (8192, 300)], [(9000, 0), (9000, 1)],
                                   [(262_144, 64), (300, 16)]])
def test_whole_requests_and_slices(api, oracle, kind, sizes):
    """Both sides of the lines between one workgroup and slices, which follow all requests of a call."""
    import torch
    g = np.random.default_rng(len(sizes) * sizes[0][0])
    score = [SCORES[kind](g, n).astype(np.float32) for n, _ in sizes]
    reqs, outs = [], []
    for s, (n, k) in zip(score, sizes):
        idx, best = torch.full((max(k, 1),), 7, dtype=torch.int32, device="cuda"), torch.zeros(max(k, 1), device="cuda")
        reqs.append(api.TopkRequest(torch.from_numpy(s).cuda(), n, k, idx, best))
        outs.append((idx, best))
    api.fs_topk(reqs)
    for s, (n, k), (idx, best) in zip(score, sizes, outs):
        e_idx, e_best = oracle.topk(s, k)
        assert np.array_equal(idx.cpu().numpy()[:k], e_idx)
        assert np.array_equal(best.cpu().numpy()[:k].view(np.uint32), e_best.view(np.uint32))
