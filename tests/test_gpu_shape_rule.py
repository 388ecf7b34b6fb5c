"""The one-series launch's own workgroups by what a wavefront has to itself against the
horizon: at the sizes around which their number changes (256 CUs), distances and
sample-days equal those of a set shape."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu
TH = np.array([0.3, 15, 0.4, 0.01, 0.4, 0.01, 0.5, 0.6], np.float32)


@pytest.mark.parametrize("T,n,flags,q", [
    (12, 7_340_032, 0, 1e-3), (12, 7_339_968, 0x20, 1e-3),                                   # four, three
    (12, 262_144, 0x8, 1e-3), (12, 262_080, 0x8, 1e-3), (12, 524_289, 0x8, 1e-3),            # raw: two, one, three
    (12, 131_073, 0, None), (12, 262_145, 0, None), (12, 524_289, 0x4, None),                # no exits: one, two, four
    (300, 3_700_000, 0, 1e-4),                                                               # a long horizon: two
])
def test_own_workgroups_equal_a_set_shape(T, n, flags, q):
    import torch
    from paper_2012_14332_amd import abc
    P = 60_000_000
    ser = abc.DeviceSeries(P, T, torch.tensor(O.observe(O.make_model(P, T), TH, 3)))
    d0 = abc.simulate_distance(ser, 50_000, 1, flags=flags)
    eps = float("inf") if q is None else float(d0.kthvalue(max(1, int(50_000 * q))).values)
    days = torch.zeros(2, dtype=torch.int64, device="cuda")
    assert abc.get_launch_config() == (0, 0, 0)
    got = abc.simulate_distance(ser, n, 7, flags=flags, eps_exit=eps, days=days[:1])
    try:
        abc.set_launch_config(1, 256, 3)
        want = abc.simulate_distance(ser, n, 7, flags=flags, eps_exit=eps, days=days[1:])
    finally:
        abc.set_launch_config(0, 0, 0)
    assert torch.equal(got, want) and int(days[0]) == int(days[1])
