"""Gradients at the batch sizes where a row kernel's last workgroup, a fragment
of 32 rows, a 64-row tile of the bias sums or a range of the weight gradients is
partly empty, against the float64 reference (bars as tests/test_gpu_mdn.py)."""
import numpy as np
import pytest

import oracle
from oracle import mdn as ref
from paper_2012_14332_amd import workloads as W
from test_gpu_mdn import A, _cos, _net_with, _rand_params, _rel  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 255, 256, 257, 511, 512, 545, 4225])
def test_gradient_at_partial_blocks(A, n):
    import torch
    rng = np.random.default_rng(n)
    feats = torch.from_numpy(rng.uniform(0, 15, size=(max(n, 2), 96)).astype(np.float32)).cuda()
    theta = oracle.prior(n, seed=4)
    p = _rand_params(3)
    net, x = _net_with(A, p, feats)
    # a larger batch first: the workspace then holds its rows past the end of this one
    net.loss_grad(torch.rand((5000, 96), device="cuda") * 15, torch.rand((5000, 8), device="cuda"))
    loss, g = net.loss_grad(feats[:n], torch.from_numpy(theta).cuda())
    again, g2 = net.loss_grad(feats[:n], torch.from_numpy(theta).cuda())
    assert torch.equal(g, g2)
    t = ref.theta_standardise(theta, W.PRIOR_LO, W.PRIOR_HI)
    loss_ref, g_ref, _ = ref.loss_and_grad(p.astype(np.float64), x[:n], t)
    assert abs(float(loss.item()) - loss_ref) <= 1e-2 * abs(loss_ref) + 1e-3
    g = g.cpu().numpy()
    assert _cos(g, g_ref) > 0.999 and _rel(g, g_ref) < 3e-2, (_cos(g, g_ref), _rel(g, g_ref))
    for part, part_ref in zip(ref.unflatten(g.astype(np.float64)), ref.unflatten(g_ref)):
        assert _cos(part, part_ref) > 0.995
    net.close()
