"""Float64 paths with parameters below zero: a negative kappa starts with a negative
count, from which nothing is drawn unless the draw itself is positive."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu
BASE = np.array([0.3, 15, 0.4, 0.01, 0.4, 0.01, 0.5, 0.6], np.float32)


def _theta():
    rows = []
    for j in range(8):
        for v in (-1e-3, -0.5, -2.0):
            rows.append(np.where(np.arange(8) == j, np.float32(v), BASE))
            # and kappa with it, so that hazards of two negative factors are positive
            rows.append(np.where((np.arange(8) == j) | (np.arange(8) == 7), np.float32(v), BASE))
    return np.array(rows + [BASE] * 16, np.float32)


@pytest.mark.parametrize("T", [1, 5, 49])
@pytest.mark.parametrize("literal", [0, 1])
def test_negative_parameters_equal_the_oracle(T, literal):
    import torch
    from paper_2012_14332_amd import abc
    P, flags = 60_000_000, abc.ABC_FP64 | (abc.ABC_NOISE_LITERAL if literal else 0)
    m = O.make_model(P, T, noise_mode=literal)
    obs = O.observe(m, BASE, 3)
    ser = abc.DeviceSeries(P, T, torch.tensor(obs))
    th = _theta()
    tg = torch.tensor(th).cuda()
    want = O.record(m, th, 5)
    small = np.abs(want).max(axis=(1, 2)) < 2**31  # counts the library holds
    got = abc.simulate_record(ser, tg, 5, flags=flags).cpu().numpy()
    assert np.array_equal(got[small], want[small])
    dist = O.distances(m, obs, 5, len(th), theta=th)
    rows = abc.simulate_rows_f64(ser, 5, torch.arange(len(th)).cuda(), tg, flags=flags & ~abc.ABC_FP64)
    full = abc.simulate_distance(ser, len(th), 5, theta=tg, flags=flags, want64=True)[1]
    for d in (rows, full):
        np.testing.assert_allclose(d.cpu().numpy()[small], dist[small], rtol=1e-12)
    eps = float(np.nanquantile(dist[small], 0.5))
    d = abc.simulate_distance(ser, len(th), 5, theta=tg, flags=flags, want64=True, eps_exit=eps)[1].cpu().numpy()
    inside = small & (dist <= np.float32(eps))
    np.testing.assert_allclose(d[inside], dist[inside], rtol=1e-12)
    assert not np.any(d[small & ~inside] <= np.float32(eps))
