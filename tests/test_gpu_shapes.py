"""Launch shapes that a kernel chooses for itself, and a launch whose observed
rows leave no room for the rings of the requested workgroup."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu
TH = np.array([0.3, 15, 0.4, 0.01, 0.4, 0.01, 0.5, 0.6], np.float32)


def _series(P, T, seed):
    import torch
    from paper_2012_14332_amd import abc
    return abc.DeviceSeries(P, T, torch.tensor(O.observe(O.make_model(P, T), TH, seed)))


# sizes at which the chosen number of workgroups per CU changes on 256 CUs (and one beyond)
@pytest.mark.parametrize("n", [1, 63, 917_503, 1_835_008, 3_670_017])
@pytest.mark.parametrize("eps,flags", [(float("inf"), 0x8), (14.0, 0), (14.0, 0x2)])
def test_own_shape_equals_a_set_shape(n, eps, flags):
    import torch
    from paper_2012_14332_amd import abc
    ser = _series(60_000_000, 12, 3)
    kw = dict(flags=flags, eps_exit=eps)
    days = torch.zeros(2, dtype=torch.int64, device="cuda")
    got = abc.simulate_distance(ser, n, 7, days=days[:1], **kw)
    try:
        abc.set_launch_config(1, 256, 3)
        want = abc.simulate_distance(ser, n, 7, days=days[1:], **kw)
    finally:
        abc.set_launch_config(0, 0, 0)
    assert torch.equal(got, want) and int(days[0]) == int(days[1])


@pytest.mark.parametrize("shape", [(0, 0, 0), (1, 1024, 1)])
def test_eight_longest_series_in_one_launch(shape):
    """131 KB of observed rows: a 1024-thread workgroup's rings do not fit beside them."""
    import torch
    from paper_2012_14332_amd import abc
    sers = [_series(5_000_000 + j, 1024, j) for j in range(8)]
    try:
        abc.set_launch_config(*shape)
        got = abc.simulate_distance_multi([{"ser": s, "n": 100 + j, "eps_exit": 30.0 if j % 2 else float("inf")}
                                           for j, s in enumerate(sers)], 5)
    finally:
        abc.set_launch_config(0, 0, 0)
    for j, s in enumerate(sers):
        want = abc.simulate_distance(s, 100 + j, 5, series=j, eps_exit=30.0 if j % 2 else float("inf"))
        assert torch.equal(got[j], want)


# round sizes at which the chosen number of workgroups per CU changes on 256 CUs
@pytest.mark.parametrize("round_size", [3_145_728, 3_145_729, 4_718_593])
@pytest.mark.parametrize("proposal", [False, True])
def test_batch_own_shape_equals_a_set_shape(round_size, proposal):
    import torch
    from paper_2012_14332_amd import abc
    sers = [_series(40_000_000 + j, 9 + 3 * j, j) for j in range(3)]
    eps = [float(abc.simulate_distance(s, 40_000, 1).kthvalue(40).values) for s in sers]
    kw = dict(max_samples=1 << 26)
    if proposal:
        rows = torch.randn((3, 136), generator=torch.Generator().manual_seed(2)) * 0.5
        kw.update(mix=rows.cuda(), lam=0.4, inflate=2.0)
    got = abc.batch_run(sers, eps, 4, 40, round_size=round_size, **kw)
    try:
        abc.set_launch_config(2, 512, 1)
        want = abc.batch_run(sers, eps, 4, 40, round_size=round_size, **kw)
    finally:
        abc.set_launch_config(0, 0, 0)
    for k in ("idx", "theta", "dist", "count", *(("w",) if proposal else ())):
        assert torch.equal(got[k], want[k]), k
    assert int(got["count"].min()) == 40
