"""Filter steps whose observation is so improbable that the sum of the belief
is a subnormal float: the steps after it must again have all their bits,
whether the step lies inside a stored segment or starts one.  Against the FP64
oracle, with the other filter sets' tolerances (test_gpu_filter_adjoint.py)."""
import numpy as np
import pytest

import oracle
from paper_1810_00204_amd import workloads as wl
from tests.test_gpu_filter_adjoint import _grad_close, _say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _far_landmark(W, H, dist, sharp, T=24):
    """Start belief a Gaussian (sigma 5) around column 12 of a map without
    walls, landmark 1 seen at step 2 `dist` cells away; with `sharp`, all four
    wall bits misread at four later steps."""
    rng = np.random.default_rng([1810, dist])
    occ = np.zeros(W * H, np.uint8)
    centre = H // 2 * W + 12
    slip = wl.slip_table_8()
    prob = wl.Problem(name="", W=W, H=H, occ=occ, slip=slip, flip=np.full(4, 0.1, np.float32),
                      lm_cell=np.array([centre + dist], np.int32), lm_p=0.8,
                      R=np.zeros((W * H, 8), np.float32), goal=-1, gamma=0.95,
                      b0=wl.belief_gaussian(occ, W, H, centre, 5.0))
    acts = rng.integers(0, 8, (1, T)).astype(np.int32)
    obs = np.zeros((1, T), np.int32)
    obs[0, 1] = 16
    if sharp:
        obs[0, 5:9] = 15
    theta = np.log(slip + 0.05).astype(np.float32)
    phi = np.array([-2.2, -1.9, -2.5, -2.0], np.float32)
    return prob, theta, phi, acts, obs


@pytest.mark.parametrize("ckpt", [2, 7])   # segments from step 2 on, and across it
@pytest.mark.parametrize("sharp", [False, True])
@pytest.mark.parametrize("W,H,dist", [
    (100, 40, 65), (100, 40, 67),          # sums of about 4e-39 and 2e-41
    (133, 133, 67)])                       # one band
def test_filter_goes_on_after_a_subnormal_sum(W, H, dist, sharp, ckpt):
    _say(f"filter {W}x{H}, landmark {dist} cells away, sharp {sharp}, segments of {ckpt}")
    from paper_1810_00204_amd.filter import FilterProblem
    prob, theta, phi, acts, obs = _far_landmark(W, H, dist, sharp)
    fp = FilterProblem(prob, acts, obs, ckpt_every=ckpt)
    nll, _, _ = fp.run(torch.as_tensor(theta), torch.as_tensor(phi))
    only, _, _ = fp.run(torch.as_tensor(theta), torch.as_tensor(phi), grad=False)
    torch.cuda.synchronize()
    onll, _, _ = oracle.filter_nll_grad(prob, theta, phi, acts, obs)
    assert onll[0] > 85
    np.testing.assert_allclose(nll.cpu().numpy(), onll, rtol=2e-5)
    assert torch.equal(nll, only)


def test_filter_gradient_across_a_tiny_sum():
    """The same with a sum that 1/eta still fits beside (about 1e-36): the
    gradient too."""
    _say("filter gradient across a tiny sum")
    from paper_1810_00204_amd.filter import FilterProblem
    prob, theta, phi, acts, obs = _far_landmark(100, 40, 62, False)
    fp = FilterProblem(prob, acts, obs, ckpt_every=7)
    nll, gs, gf = fp.run(torch.as_tensor(theta), torch.as_tensor(phi))
    torch.cuda.synchronize()
    onll, ogt, ogp = oracle.filter_nll_grad(prob, theta, phi, acts, obs)
    np.testing.assert_allclose(nll.cpu().numpy(), onll, rtol=2e-5)
    _grad_close(np.concatenate([gs.cpu().numpy().ravel(), gf.cpu().numpy()]),
                np.concatenate([ogt.ravel(), ogp]))
