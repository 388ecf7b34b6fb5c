"""A quota run whose last rounds are the last its limit allows: a small
candidate capacity makes many short rounds."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("quota", [20, 59, 65, 71])
@pytest.mark.parametrize("behind", [2, 4])
def test_quota_met_in_the_last_rounds(quota, behind):
    import torch
    from paper_2012_14332_amd import abc, pipeline as P, workloads as W
    ser = P.observed_series(W.uneven_series(64, 5)[0])
    eps = P.pilot_eps(ser, 9, n=20_000, q=1e-2, series=0)
    want = abc.batch_run([ser], [eps], 9, quota, round_size=1 << 14)
    got = abc.batch_run([ser], [eps], 9, quota, round_size=1 << 22, max_samples=1 << 17, cand_capacity=130,
                        rounds_per_graph=behind)
    for key in ("idx", "theta", "dist", "count", "mean", "cov"):
        assert torch.equal(got[key], want[key])
