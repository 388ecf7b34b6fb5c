"""ABC-SMC generations at population sizes around the chunks of the ordered
sums, with and without the float64 band, against the oracle (bars as
tests/test_gpu_smc.py); the stable compaction of decided rows across its steps."""
import numpy as np
import pytest

from oracle import smc as osmc
from test_gpu_smc import _compare, _upload, env  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [15, 17, 127, 128, 129, 143, 144, 145, 257])
@pytest.mark.parametrize("band_w", [0.02, 0.0])
def test_population_sizes_around_a_chunk(env, N, band_w):
    abc, s, m, obs, eps0, ser = env
    prev = osmc.smc_abc(m, obs, seed=6, N=N, generations=1, alpha=0.5, eps0=eps0)[0]
    cfg = abc.smc_config(N, eps0, alpha=0.5, chunk0=1 << 12, chunk_max=1 << 14, band_w=band_w)
    out = abc.smc_generation(ser, cfg, 6, 1, _upload(prev), want_ancestors=True)
    if band_w:
        _compare(out, osmc.smc_abc(m, obs, seed=6, N=N, generations=2, alpha=0.5, eps0=eps0)[1], "gen1")
        return
    # without a band float32 decides; everything that follows from the rows is as defined
    idx, th, anc = (out[k].cpu().numpy() for k in ("idx", "theta", "ancestors"))
    mean, cov = osmc.weighted_mean_cov(prev.theta, prev.W)
    L = osmc.cholesky(2.0 * cov)
    u, z = osmc.proposal_draws(6, 0, 1, 0, int(idx[-1]) + 1)
    anc_all, th_all = osmc.perturb(prev.theta, osmc.cumulative(prev.W), L, u, z)
    np.testing.assert_array_equal(th, th_all[idx])
    np.testing.assert_array_equal(anc, anc_all[idx])
    d = abc.simulate_rows_f64(ser, 6, out["idx"], out["theta"], domain=7, series=1 << 16)
    import torch
    assert torch.equal(d, out["dist"]) and out["stats"]["samples"] == idx[-1] + 1
    w = osmc.normalise(osmc.kernel_weights(th, prev.theta, prev.W, 2.0 * cov))
    got = out["w"].cpu().numpy()
    assert np.max(np.abs(got - w) / w) <= 1e-10


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 2048, 5000])
@pytest.mark.parametrize("weighted", [False, True])
def test_decided_rows_stay_in_order(env, n, weighted):
    import torch
    abc, s, m, obs, eps0, ser = env
    d = abc.simulate_distance(ser, n, 3)
    eps = float(d.median())
    # rows up to twice eps, decided in float64 above half of it: every step drops some
    w_all = torch.arange(n, device="cuda", dtype=torch.float32) if weighted else None
    idx, th, dist, w, count = abc.accept_compact(d, 2 * eps, n, seed=3, weight=w_all)
    c = int(count)
    i0, t0, d0 = idx[:c].clone(), th[:c].clone(), dist[:c].clone()
    d64 = abc.simulate_rows_f64(ser, 3, i0, t0)
    band = (d0 > np.float32(eps * 0.5)) & (d0 <= np.float32(eps * 1.5))
    keep = torch.where(band, d64 <= np.float32(eps), d0 <= eps)
    abc.recheck_band(ser, 3, eps, 0.5, idx, th, dist, count, weight=w)
    k = int(count)
    assert k == int(keep.sum())
    assert torch.equal(idx[:k], i0[keep]) and torch.equal(th[:k], t0[keep])
    assert torch.equal(dist[:k], torch.where(band, d64.float(), d0)[keep])
    if weighted:
        assert torch.equal(w[:k], i0[keep].float())
