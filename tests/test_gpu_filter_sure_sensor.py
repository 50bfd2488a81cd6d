"""Flip gradients of a sensor that is almost always right, or almost always
wrong: the few misread (rightly read) cells' share must keep its own digits.
Against the FP64 oracle, with the other filter sets' tolerances
(test_gpu_filter_adjoint.py).

f = 1 - 2^-20 is a float, and so are the kernel's steps to it from phi =
log(2^20 - 1); other flips near 1 differ from the oracle's by their rounding."""
import numpy as np
import pytest

import oracle
from paper_1810_00204_amd import workloads as wl
from tests.test_gpu_filter_adjoint import _grad_close, _say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("W,H", [(24, 24), (40, 17)])
@pytest.mark.parametrize("phi", [(-13.0, -12.0, -12.5, -13.5), (-15.0, -15.5, -14.5, -15.0),
                                 (np.log(2.0 ** 20 - 1.0),) * 4])
def test_filter_flip_gradient_of_a_sure_sensor(W, H, phi):
    _say(f"filter {W}x{H}, phi {phi[0]:.1f}")
    from paper_1810_00204_amd.filter import FilterProblem
    phi = np.asarray(phi, np.float32)
    rng = np.random.default_rng([1810, W, H, int(abs(phi[0]))])
    occ = wl.occ_exact_count(rng, W, H, 0.15)
    free = np.flatnonzero(occ == 0)
    slip = wl.slip_table_8()
    flip = (1 / (1 + np.exp(-phi.astype(np.float64)))).astype(np.float32)
    acts = rng.integers(0, 8, (6, 40)).astype(np.int32)
    obs = np.stack([wl._simulate(rng, occ, W, H, slip, flip, int(rng.choice(free)), a,
                                 np.zeros(W * H, np.int32), 0.8) for a in acts]).astype(np.int32)
    prob = wl.Problem(name="", W=W, H=H, occ=occ, slip=slip, flip=flip,
                      lm_cell=np.zeros(0, np.int32), lm_p=0.8, R=np.zeros((W * H, 8), np.float32),
                      goal=-1, gamma=0.95, b0=wl.belief_uniform_cells(W * H, free))
    theta = (np.log(slip + 0.05) + rng.normal(0, 0.4, slip.shape)).astype(np.float32)
    fp = FilterProblem(prob, acts, obs, ckpt_every=7)
    nll, gs, gf = fp.run(torch.as_tensor(theta), torch.as_tensor(phi))
    torch.cuda.synchronize()
    onll, ogt, ogp = oracle.filter_nll_grad(prob, theta, phi, acts, obs)
    np.testing.assert_allclose(nll.cpu().numpy(), onll, rtol=2e-5)
    _grad_close(np.concatenate([gs.cpu().numpy().ravel(), gf.cpu().numpy()]),
                np.concatenate([ogt.ravel(), ogp]))
