"""Training pairs of short horizons, on both sides of the longest one from which a large
call orders its samples: the values of calls too small to be ordered."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,T_lo,T_hi", [(9000, 1, 3), (20_001, 5, 39), (20_001, 5, 40)])
def test_large_calls_equal_small_ones(n, T_lo, T_hi):
    import torch
    from paper_2012_14332_amd import abc
    kw = dict(T_lo=T_lo, T_hi=T_hi)
    whole = abc.simulate_features(n, 11, first=5, **kw)
    parts = [abc.simulate_features(min(5000, n - a), 11, first=5 + a, **kw) for a in range(0, n, 5000)]
    for k in range(3):
        assert torch.equal(whole[k], torch.cat([p[k] for p in parts]))
