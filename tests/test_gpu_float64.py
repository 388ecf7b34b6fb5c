"""Float64 paths at the edges of their own arithmetic: exponents inside, at and
beyond the range of the short power (n = 16), the row kernels' group sizes, and
horizons around their windows, against the oracle."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


def _theta(n, seed):
    rng = np.random.default_rng(seed)
    th = (rng.random((n, 8)) * np.array([1, 100, 2, 1, 1, 1, 1, 2])).astype(np.float32)
    th[:, 2] = np.resize(np.array([0, 0.5, 1, 2, 15.75, 16, 16.25, 60, 200], np.float32), n)
    th[::7, 4] = 0.0   # no recovery: M stays at A0 + R0 + D0
    th[::11, 3] = 0.0
    return th


# trajectories are integers: equal unless a draw lies within the arithmetic's
# error (about 1e-12 of a count) of an integer
@pytest.mark.parametrize("P,T,A0", [(1000, 33, 1), (60_000_000, 64, 100), (2_000_000_000, 65, 3)])
def test_record_at_exponent_edges(P, T, A0):
    import torch
    from paper_2012_14332_amd import abc
    th = _theta(90, T)
    ser = abc.DeviceSeries(P, T, A0=A0)
    got = abc.simulate_record(ser, torch.tensor(th, device="cuda"), 5, flags=abc.ABC_FP64).cpu().numpy()
    want = O.record(O.make_model(P, T, A0=A0), th, 5)
    assert np.array_equal(got, want)


# distances: float64 sums of at most 3 T terms, each a few ulp
@pytest.mark.parametrize("n", [1, 3, 256, 257, 1024, 4097, 16500])
@pytest.mark.parametrize("T,flags", [(1, 0), (31, 0x8), (33, 0x4)])
def test_rows_equal_the_sample_kernel_and_the_oracle(n, T, flags):
    import torch
    from paper_2012_14332_amd import abc
    obs = O.observe(O.make_model(5_000_000, T), np.array([0.3, 15, 0.4, 0.01, 0.4, 0.01, 0.5, 0.6], np.float32), 9)
    ser = abc.DeviceSeries(5_000_000, T, torch.tensor(obs))
    th = torch.tensor(_theta(n, 1), device="cuda")
    idx = torch.arange(7, 7 + n, device="cuda")
    rows = abc.simulate_rows_f64(ser, 3, idx, th, flags=flags)
    _, d64 = abc.simulate_distance(ser, n, 3, theta=th, first=7, flags=flags | abc.ABC_FP64, want64=True)
    assert torch.equal(rows, d64)
    m = O.make_model(5_000_000, T, noise_mode=1 if flags & 0x4 else 0, dist_mode=1 if flags & 0x8 else 0)
    k = min(n, 500)
    want = O.distances(m, obs, 3, k, first=7, theta=th[:k].cpu().numpy())
    np.testing.assert_allclose(rows[:k].cpu().numpy(), want, rtol=1e-12)


@pytest.mark.parametrize("T", [40, 96, 200])
def test_exit_bound_changes_no_distance(T):
    """With the bound on the days still to come an early exit ends the same samples."""
    import torch
    from paper_2012_14332_amd import abc
    obs = O.observe(O.make_model(5_000_000, T), np.array([0.3, 15, 0.4, 0.01, 0.4, 0.01, 0.5, 0.6], np.float32), 9)
    ser = abc.DeviceSeries(5_000_000, T, torch.tensor(obs))
    _, full = abc.simulate_distance(ser, 4000, 3, flags=abc.ABC_FP64, want64=True)
    eps = float(np.quantile(full.cpu().numpy(), 0.02).astype(np.float32))
    for flags in (0, abc.ABC_NO_BOUND):
        _, d = abc.simulate_distance(ser, 4000, 3, flags=abc.ABC_FP64 | flags, want64=True, eps_exit=eps)
        inside = full <= eps
        assert torch.equal(d[inside], full[inside]) and bool(torch.isinf(d[~inside]).all())


@pytest.mark.parametrize("n", [1, 3, 64, 700, 5000, 40_000])
@pytest.mark.parametrize("T", [7, 33, 49, 300])
@pytest.mark.parametrize("flags", [0x1, 0x1 | 0x8, 0x1 | 0x4])
def test_last_samples_walked_as_rows(n, T, flags):
    """Exits leave few samples to a wavefront, which then walks them again side by
    side: same distances as a pass without exits, infinite past the bound."""
    import torch
    from paper_2012_14332_amd import abc
    P = 60_000_000
    obs = O.observe(O.make_model(P, T), np.array([0.3, 15, 0.4, 0.01, 0.4, 0.01, 0.5, 0.6], np.float32), 4)
    ser = abc.DeviceSeries(P, T, torch.tensor(obs))
    full = abc.simulate_distance(ser, n, 11, flags=flags, want64=True)[1]
    for q in (0.0, 0.02, 0.5, 1.0):
        eps = float(torch.quantile(full, q))
        d32, got = abc.simulate_distance(ser, n, 11, flags=flags, eps_exit=eps, want64=True)
        inside = full <= float(np.float32(eps))
        assert torch.equal(got[inside], full[inside]), (q, n)
        # beyond the tolerance a sample is either ended or finished
        assert torch.all(torch.isinf(got[~inside]) | (got[~inside] == full[~inside]))
        assert torch.equal(d32, got.float())
