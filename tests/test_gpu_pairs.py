"""Training pairs and their standardisation: the ordered launch against the
unordered one, and the column statistics at the edges of their row ranges."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,T_lo,T_hi", [(8192, 30, 200), (33001, 1, 40), (20000, 7, 1024), (8193, 50, 51)])
def test_ordered_pairs_equal_unordered(n, T_lo, T_hi):
    """A large call orders its samples by horizon; calls below 8192 do not. Same values."""
    import torch
    from paper_2012_14332_amd import abc
    kw = dict(T_lo=T_lo, T_hi=T_hi)
    whole = abc.simulate_features(n, 11, first=5, **kw)
    parts = [abc.simulate_features(min(5000, n - a), 11, first=5 + a, **kw) for a in range(0, n, 5000)]
    for k in range(3):
        assert torch.equal(whole[k], torch.cat([p[k] for p in parts]))


# float64 sums of n terms rounded to float32 once: half an ulp (6e-8), with room for the last bit
@pytest.mark.parametrize("n", [2, 3, 79, 80, 81, 8000, 81921, 100003])
@pytest.mark.parametrize("aligned", [True, False])
def test_column_statistics(n, aligned):
    import torch
    from paper_2012_14332_amd import abc
    x = (np.random.default_rng(n).standard_normal((n, 96)) * 0.01 + np.arange(96)).astype(np.float32)
    x[:, 5] = 3.25
    buf = torch.empty(n * 96 + 1, dtype=torch.float32, device="cuda")
    f = (buf[:-1] if aligned else buf[1:]).view(n, 96)
    f.copy_(torch.tensor(x))
    net = abc.Mdn(0)
    net.fit_standardizer(f)
    m, s = (t.cpu().numpy() for t in net.standardizer())
    x = x.astype(np.float64)
    np.testing.assert_allclose(m, x.mean(0), rtol=1.2e-7, atol=1e-12)
    np.testing.assert_allclose(s, np.maximum(x.std(0, ddof=1), 1e-6), rtol=1.2e-7)


def test_pairs_and_statistics_in_a_captured_graph():
    """Captured calls take no scratch of the library's; each replay gives the eager call's values."""
    import torch
    from paper_2012_14332_amd import abc
    want = abc.simulate_features(9001, 11, first=5)
    net = abc.Mdn(0)
    net.fit_standardizer(want[0])
    stats = net.standardizer()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = abc.simulate_features(9001, 11, first=5)
        net.fit_standardizer(got[0])
        got_stats = net.standardizer()
    for _ in range(3):
        for t in got + got_stats:
            t.zero_()
        abc.simulate_features(20000, 3)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(got + got_stats, want + stats):
            assert torch.equal(a, b)
