"""The multi-series launch's own workgroups where a job has no early exit, or a raw
distance: at the sizes around which their number changes (256 CUs), distances and
sample-days equal those of a set shape."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu
TH = np.array([0.3, 15, 0.4, 0.01, 0.4, 0.01, 0.5, 0.6], np.float32)


@pytest.mark.parametrize("Ts,n,flags,exits", [
    ((9, 14, 12), 43_000, 0, "none"), ((9, 14, 12), 90_000, 0, "some"), ((9, 14, 12), 175_000, 0, "none"),
    ((9, 14, 12), 90_000, 0x8, "all"), ((9, 200, 12), 90_000, 0x8, "all"), ((9, 14, 12), 1_300_000, 0, "all"),
])
def test_own_workgroups_equal_a_set_shape(Ts, n, flags, exits):
    import torch
    from paper_2012_14332_amd import abc
    P = 60_000_000
    sers = [abc.DeviceSeries(P, T, torch.tensor(O.observe(O.make_model(P, T), TH, T))) for T in Ts]
    eps = [float(abc.simulate_distance(s, 20_000, 1, flags=flags).kthvalue(40).values) for s in sers]
    jobs = [{"ser": s, "n": n + 5 * j, "eps_exit": e if exits == "all" or (exits == "some" and j == 1) else float("inf")}
            for j, (s, e) in enumerate(zip(sers, eps))]
    days = torch.zeros(2, dtype=torch.int64, device="cuda")
    assert abc.get_launch_config() == (0, 0, 0)
    got = abc.simulate_distance_multi(jobs, 7, flags=flags, days=days[:1])
    try:
        abc.set_launch_config(1, 256, 3)
        want = abc.simulate_distance_multi(jobs, 7, flags=flags, days=days[1:])
    finally:
        abc.set_launch_config(0, 0, 0)
    for a, b in zip(got, want):
        assert torch.equal(a, b)
    assert exits != "none" or int(days[0]) == int(days[1]) == sum(j["n"] * j["ser"].T for j in jobs)
