"""Selection and compaction at the sizes where a step is partly filled: the
nearest k of row sets that one workgroup holds or not, of candidate sets on
both sides of the counted ranks, over several histogram passes; compaction of a
last step of every length; moments of a few rows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _dists(kind, n, rng):
    d = rng.lognormal(3.0, 1.0, n).astype(np.float32)
    if kind == "ties":
        d = np.round(d)
    elif kind == "same":
        d[:] = 7.0
    elif kind == "odd":
        d[:: 3] = np.inf
        d[1:: 7] = np.nan
        d[2] = -0.0
    elif kind == "far":  # most rows in one bin of the first pass
        d = (1.0 + rng.random(n) * 1e-3).astype(np.float32)
        d[0] = 1e30
    return d


@pytest.mark.parametrize("kind", ["plain", "ties", "same", "odd", "far"])
@pytest.mark.parametrize("n,k", [(5, 1), (1023, 300), (1024, 511), (1025, 512), (4097, 513), (40_000, 4096), (70_001, 100)])
def test_nearest_k(n, k, kind):
    import torch
    from paper_2012_14332_amd import abc
    d = _dists(kind, n, np.random.default_rng(n + k))
    idx, th, dd, kth = abc.nearest_k(torch.tensor(d).cuda(), k, first=5, seed=2)
    order = np.lexsort((np.arange(n), np.where(np.isnan(d), np.inf, d) + 0.0))[:k]
    want = np.sort(order)
    assert np.array_equal(idx.cpu().numpy(), want + 5)
    assert np.array_equal(dd.cpu().numpy(), d[want])
    assert float(kth) == d[order[-1]]
    assert torch.equal(th, abc.sample_prior(n, seed=2, first=5)[torch.tensor(want).cuda()])


def test_nearest_k_of_too_few_finite():
    import torch
    from paper_2012_14332_amd import abc
    d = torch.full((5000,), float("inf"), device="cuda")
    d[:9] = 1.0
    with pytest.raises(abc.AbcError, match="only 9 of the 5000"):
        abc.nearest_k(d, 10, seed=2)


@pytest.mark.parametrize("n,k", [(1, 1), (7, 3), (8, 8), (9, 4), (1023, 1023), (1024, 77), (1025, 77)])
@pytest.mark.parametrize("kind", ["plain", "ties", "odd"])
def test_nearest_k_rows(n, k, kind):
    import torch
    from paper_2012_14332_amd import abc
    rng = np.random.default_rng(n)
    d = _dists(kind, max(n, 3), rng)[:n].astype(np.float64)
    i = rng.permutation(10 * n)[:n].astype(np.int64)
    th = rng.random((n, 8)).astype(np.float32)
    idx, t, dd = abc.nearest_k_rows(torch.tensor(d).cuda(), torch.tensor(i).cuda(), torch.tensor(th).cuda(), k)
    order = np.lexsort((i, d, np.isnan(d)))[:k]
    want = order[np.argsort(i[order])]
    assert np.array_equal(idx.cpu().numpy(), i[want])
    assert np.array_equal(t.cpu().numpy(), th[want])
    assert np.array_equal(dd.cpu().numpy(), d[want], equal_nan=True)


@pytest.mark.parametrize("n", [9, 1025])
def test_nearest_k_rows_of_one_index(n):
    """Rows that share the largest index: only kept rows count for a kept row's place."""
    import torch
    from paper_2012_14332_amd import abc
    d = np.arange(n, 0, -1).astype(np.float64)
    i = np.full(n, np.iinfo(np.int64).max)
    th = torch.zeros((n, 8), device="cuda")
    idx, _, dd = abc.nearest_k_rows(torch.tensor(d).cuda(), torch.tensor(i).cuda(), th, 4)
    assert np.array_equal(idx.cpu().numpy(), i[:4]) and dd.cpu().tolist() == [4.0, 3.0, 2.0, 1.0]


@pytest.mark.parametrize("n", [1, 3, 63, 1023, 1024, 4095, 4096, 4097, 8191, 65_537])
def test_compaction_of_a_partial_step(n):
    import torch
    from paper_2012_14332_amd import abc
    d = np.random.default_rng(n).random(n).astype(np.float32)
    d[-1] = 0.5
    idx, th, dd, _, count = abc.accept_compact(torch.tensor(d).cuda(), 0.5, n, seed=3)
    want = np.nonzero(d <= 0.5)[0]
    c = int(count)
    assert np.array_equal(idx[:c].cpu().numpy(), want) and np.array_equal(dd[:c].cpu().numpy(), d[want])


@pytest.mark.parametrize("n", [0, 1, 2, 5, 63, 64, 65, 255, 256, 257, 2049])
@pytest.mark.parametrize("weighted", [False, True])
def test_moments_of_a_few_rows(n, weighted):
    import torch
    from paper_2012_14332_amd import abc
    rng = np.random.default_rng(n)
    th = rng.random((max(n, 1), 8)).astype(np.float32)[:n]
    w = (rng.random(n) + 0.1).astype(np.float32) if weighted else np.ones(n, np.float32)
    mean, cov = abc.posterior_moments(torch.tensor(th).cuda(), weight=torch.tensor(w).cuda() if weighted else None)
    mean, cov = mean.cpu().numpy(), cov.cpu().numpy()
    if n == 0:
        assert np.all(np.isnan(mean)) and np.all(np.isnan(cov))
        return
    x, v = th.astype(np.float64), w.astype(np.float64)
    m = (v[:, None] * x).sum(0) / v.sum()
    # a few hundred additions of numbers below one in float64
    assert np.max(np.abs(mean - m)) <= 1e-13
    if n == 1:
        assert np.all(np.isnan(cov))
        return
    c = x - m
    want = (v[:, None, None] * c[:, :, None] * c[:, None, :]).sum(0) / (v.sum() - (v * v).sum() / v.sum())
    assert np.max(np.abs(cov - want)) <= 1e-12 and np.array_equal(cov, cov.T)


# a unit of one step, of two, and of the most; accepts none, few and more than its kept offsets
@pytest.mark.parametrize("n", [16_777_216, 16_777_217, 40_000_001, 300_000_000])
@pytest.mark.parametrize("q", [0.0, 1e-5, 1e-3])
def test_compaction_units(n, q):
    import torch
    from paper_2012_14332_amd import abc
    d = torch.rand(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(n))
    d[n // 3: n // 3 + 9000] = 0.0 if q else 0.5  # a run of accepts across steps
    idx, _, dd, _, count = abc.accept_compact(d, q, 1 << 20, seed=3)
    want = torch.nonzero(d <= q).flatten()
    c = int(count)
    assert c == want.numel() and torch.equal(idx[:c], want) and torch.equal(dd[:c], d[want])
