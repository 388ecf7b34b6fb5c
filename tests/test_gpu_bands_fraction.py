"""Fraction of a quantile between two order statistics: (n - 1) q - floor, of the
exact product, so that a quantile whose rounded product is a whole number still
leans to the side of the exact one. Compared bit for bit."""
from fractions import Fraction

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _bands(x, qs):
    """float32 [nq][days][6]: sorted values, every step rounded as a fused operation."""
    n = x.shape[0]
    v = np.sort(x, axis=0)
    out = np.empty((len(qs),) + x.shape[1:], np.float32)
    for k, q in enumerate(qs):
        lo = min(int(np.floor(np.float64(n - 1) * np.float64(q))), n - 1)
        hi = min(lo + 1, n - 1)
        t = Fraction(float(Fraction(n - 1) * Fraction(float(q)) - lo))
        for ix in np.ndindex(*x.shape[1:]):
            a, b = int(v[(lo,) + ix]), int(v[(hi,) + ix])
            out[(k,) + ix] = np.float32(float(Fraction(b - a) * t + a))
    return out


@pytest.mark.parametrize("n", [2, 10, 64, 65, 256, 257, 512, 513, 1000, 1025, 2048, 4096, 8192])
@pytest.mark.parametrize("kind", ["few", "edge"])
def test_fraction_of_the_exact_product(n, kind):
    import torch
    from paper_2012_14332_amd import abc
    g = np.random.default_rng(n)
    if kind == "few":
        x = g.integers(0, 5, (n, 3, 6)).astype(np.int32)
    else:
        x = np.array([-2**31, 2**31 - 1, 0, 1], np.int64)[g.integers(0, 4, (n, 3, 6))].astype(np.int32)
    qs = [k / 15 for k in range(16)]
    got = abc.trajectory_bands(torch.from_numpy(x).cuda(), qs).cpu().numpy()
    assert np.array_equal(got, _bands(x, qs))
