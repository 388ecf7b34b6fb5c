"""Quantile bands at the edges of the values a lane holds, with ties and the
whole int32 range, and recording with the noise drawn apart from the walk."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _values(kind, n, T, rng):
    if kind == "wide":
        x = rng.integers(-2**31, 2**31, (n, T + 1, 6))
        x[:: max(1, n // 5)] = -2**31
        x[1:: max(1, n // 5)] = 2**31 - 1
        return x
    if kind == "ties":
        return rng.integers(0, 4, (n, T + 1, 6)) * 1000
    return np.floor(np.exp(rng.normal(9.0, 3.0, (n, T + 1, 6)))).clip(max=2**31 - 1)


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 1024, 1025, 2048, 2049, 4096, 4097, 8191, 8192])
@pytest.mark.parametrize("kind", ["wide", "ties", "spread"])
def test_bands_equal_sorted_interpolation(n, kind):
    import torch
    from paper_2012_14332_amd import abc
    rng = np.random.default_rng(n)
    T = 2
    tr = _values(kind, n, T, rng).astype(np.int32)
    for q in ((0.5,), (0.0, 1.0), (0.05, 0.5, 0.95), tuple(rng.uniform(0, 1, 16))):
        got = abc.trajectory_bands(torch.tensor(tr).cuda(), q).cpu().numpy()
        v = np.sort(tr.astype(np.float64), axis=0)
        h = (n - 1) * np.array(q)
        lo = np.minimum(np.floor(h).astype(int), n - 1)
        hi = np.minimum(lo + 1, n - 1)
        t = (h - lo)[:, None, None]
        want = v[lo] + (v[hi] - v[lo]) * t
        # one rounding to float32, and float64 sums of numbers below 2^32
        assert np.all(np.abs(got - want) <= 2.0**-24 * np.abs(want) + 2.0**-19), (q, np.abs(got - want).max())


@pytest.mark.parametrize("T", [1, 5, 6, 7, 13, 49])
@pytest.mark.parametrize("flags", [0, 0x4])  # the second: noise read literally
def test_recording_of_few_rows_equals_recording_of_many(T, flags):
    import torch
    from paper_2012_14332_amd import abc
    many = 64 * 2 * torch.cuda.get_device_properties(0).multi_processor_count + 1
    th = torch.rand((many, 8), generator=torch.Generator().manual_seed(T))
    th = (th * torch.tensor([1.0, 100, 2, 1, 1, 1, 1, 2])).cuda()
    ser = abc.DeviceSeries(60_000_000, T, A0=155, R0=2, D0=3)
    want = abc.simulate_record(ser, th, 5, first=9, flags=flags)
    for n in (1, 63, 64, 65, many - 1):
        assert torch.equal(abc.simulate_record(ser, th[:n].contiguous(), 5, first=9, flags=flags), want[:n]), n
