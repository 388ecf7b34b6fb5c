"""Column statistics where the rows differ most from the first one, and at the edges of
the row ranges."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _within(got, want, ulps):
    """float32 `got` within `ulps` half units of float32 of the float64 `want`"""
    want = np.asarray(want)
    return np.all(np.abs(got.astype(np.float64) - want) <= ulps * 2.0**-24 * np.abs(want) * (1 + 1e-6))


def test_one_row_unlike_all_others():
    """sd = |x0 - b| / sqrt(n): sums about the first row cancel n of n + 1 parts."""
    import torch
    from paper_2012_14332_amd import abc
    n = 10_000_000
    rng = np.random.default_rng(4)
    x0, b = (rng.normal(size=96) * 20).astype(np.float32), (rng.normal(size=96) * 3).astype(np.float32)
    f = torch.from_numpy(b).cuda().repeat(n, 1)
    f[0] = torch.from_numpy(x0).cuda()
    net = abc.Mdn(1)
    net.fit_standardizer(f)
    mean, sd = (t.cpu().numpy() for t in net.standardizer())
    x0, b = x0.astype(np.float64), b.astype(np.float64)
    assert _within(mean, b + (x0 - b) / n, 1)
    assert _within(sd, np.abs(x0 - b) / np.sqrt(n), 1)


@pytest.mark.parametrize("n", [2, 3, 255, 257, 4096, 4097, 4161, 81_920, 81_921, 82_900])
@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("first", [0.0, 1e6])
def test_range_edges_and_a_far_first_row(n, aligned, first):
    import torch
    from paper_2012_14332_amd import abc
    x = (torch.randn((n, 96), generator=torch.Generator().manual_seed(n)) * 3 + 5).numpy()
    x[0] += np.float32(first)
    x[:, 7] = 0.25
    buf = torch.empty(96 * n + 4, device="cuda")
    f = buf[(0 if aligned else 1):][:96 * n].view(n, 96)
    f.copy_(torch.from_numpy(x))
    net = abc.Mdn(1)
    net.fit_standardizer(f)
    mean, sd = (t.cpu().numpy() for t in net.standardizer())
    d = x.astype(np.float64)
    assert np.all(np.abs(mean - d.mean(axis=0)) <= 2.0**-24 * np.abs(d.mean(axis=0)) + 1e-12)
    assert _within(sd, np.maximum(d.std(axis=0, ddof=1), 1e-6), 1)
