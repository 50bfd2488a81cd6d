"""Gradient of runs of thousands of equal steps: the belief settles, so every
step rounds its sum the same way, and no step may hand its error on.

Tolerance: a step's terms are off by at most about 40 roundings of 2^-24
(products, the 3x3 sums, lane and wavefront sums), and an error of the
adjoint's shape dies out within a few steps (four here): 1e-5."""
import numpy as np
import pytest

import oracle
from paper_1810_00204_amd import workloads as wl
from tests.test_gpu_filter_adjoint import _grad_close, _say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _equal_steps(W, H, T, seed):
    rng = np.random.default_rng([1810, W, H, seed])
    occ = wl.occ_exact_count(rng, W, H, 0.15)
    free = np.flatnonzero(occ == 0)
    slip = wl.slip_table_8()
    prob = wl.Problem(name="", W=W, H=H, occ=occ, slip=slip, flip=np.full(4, 0.1, np.float32),
                      lm_cell=np.zeros(0, np.int32), lm_p=0.8, R=np.zeros((W * H, 8), np.float32),
                      goal=-1, gamma=0.95, b0=wl.belief_uniform_cells(W * H, free))
    acts = np.full((1, T), seed % 8, np.int32)
    obs = np.full((1, T), rng.integers(0, 16), np.int32)
    theta = (np.log(slip + 0.05) + rng.normal(0, 0.4, slip.shape)).astype(np.float32)
    return prob, theta, rng.normal(-2.0, 0.3, 4).astype(np.float32), acts, obs


@pytest.mark.parametrize("W,H,seed", [(12, 9, 0), (12, 9, 3), (16, 16, 4), (33, 20, 6)])
def test_filter_gradient_does_not_drift(W, H, seed):
    _say(f"filter drift {W}x{H} seed {seed}")
    from paper_1810_00204_amd.filter import FilterProblem
    prob, theta, phi, acts, obs = _equal_steps(W, H, 4000, seed)
    fp = FilterProblem(prob, acts, obs, ckpt_every=60)
    nll, gs, gf = fp.run(torch.as_tensor(theta), torch.as_tensor(phi))
    torch.cuda.synchronize()
    onll, ogt, ogp = oracle.filter_nll_grad(prob, theta, phi, acts, obs)
    np.testing.assert_allclose(nll.cpu().numpy(), onll, rtol=2e-5)
    _grad_close(np.concatenate([gs.cpu().numpy().ravel(), gf.cpu().numpy()]),
                np.concatenate([ogt.ravel(), ogp]), rel=1e-5, entry=1e-5)
