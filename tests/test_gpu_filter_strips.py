"""The filter kernel's strips: strips of 1, 2, 4, 12, 16 and 22 cells, both
directions, remainders of strips and of wavefronts, one band and two, with and
without a goal and landmarks, and more steps than one chunk of inputs, against
the FP64 oracle.

Tolerances as for the other filter sets (test_gpu_filter_adjoint.py): 2e-5
relative on the NLL; 1e-4 on each part and entry of the gradient, 5e-4 on
runs of hundreds of steps."""
import numpy as np
import pytest

import oracle
from paper_1810_00204_amd import workloads as wl
from tests.test_gpu_filter_adjoint import _grad_close, _say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _set(W, H, ntraj, T, L=0, goal=False, seed=0):
    rng = np.random.default_rng([1810, W, H, T, seed])
    occ = wl.occ_exact_count(rng, W, H, 0.15)
    free = np.flatnonzero(occ == 0)
    slip = wl.slip_table_8()
    lm = np.sort(rng.choice(free, size=L, replace=False)).astype(np.int32)
    lm_id = np.zeros(W * H, np.int32)
    lm_id[lm] = np.arange(1, L + 1)
    flip = np.array([0.1, 0.15, 0.07, 0.12], np.float32)
    acts = rng.integers(0, 8, (ntraj, T)).astype(np.int32)
    obs = np.stack([wl._simulate(rng, occ, W, H, slip, flip, int(rng.choice(free)), a, lm_id, 0.8)
                    for a in acts]).astype(np.int32)
    prob = wl.Problem(name="", W=W, H=H, occ=occ, slip=slip, flip=flip, lm_cell=lm, lm_p=0.8,
                      R=np.zeros((W * H, 8), np.float32),
                      goal=int(free[free.size // 2]) if goal else -1, gamma=0.95,
                      b0=wl.belief_uniform_cells(W * H, free))
    theta = (np.log(slip + 0.05) + rng.normal(0, 0.4, slip.shape)).astype(np.float32)
    phi = rng.normal(-2.0, 0.3, 4).astype(np.float32)
    return prob, theta, phi, acts, obs


@pytest.mark.parametrize("W,H,ntraj,T,ckpt,L,goal", [
    (3, 2, 2, 5, 2, 0, False),          # one wavefront, strips of 1
    (7, 40, 3, 9, 4, 3, True),
    (40, 7, 3, 9, 4, 3, True),          # the same map sizes, strips along x
    (63, 33, 3, 7, 7, 0, False),
    (33, 70, 3, 7, 3, 20, False),
    (100, 90, 2, 6, 3, 0, True),
    (128, 128, 2, 5, 2, 0, False),
    (128, 127, 2, 5, 2, 40, True),
    (1617, 10, 2, 4, 2, 0, False),      # one band, strips of 16
    (133, 133, 2, 4, 3, 5, True),       # one band, strips of 22
    (133, 133, 2, 4, 3, 0, False),
    (12, 9, 2, 600, 37, 4, False),      # several chunks of steps
])
def test_filter_strips_match_oracle(W, H, ntraj, T, ckpt, L, goal):
    _say(f"filter strips {W}x{H} T{T} L{L} goal {goal}")
    from paper_1810_00204_amd.filter import FilterProblem
    prob, theta, phi, acts, obs = _set(W, H, ntraj, T, L, goal)
    fp = FilterProblem(prob, acts, obs, ckpt_every=ckpt)
    nll, gs, gf = fp.run(torch.as_tensor(theta), torch.as_tensor(phi))
    only, _, _ = fp.run(torch.as_tensor(theta), torch.as_tensor(phi), grad=False)
    torch.cuda.synchronize()
    onll, ogt, ogp = oracle.filter_nll_grad(prob, theta, phi, acts, obs)
    np.testing.assert_allclose(nll.cpu().numpy(), onll, rtol=2e-5)
    assert torch.equal(nll, only)
    tol = 5e-4 if T > 100 else 1e-4
    _grad_close(np.concatenate([gs.cpu().numpy().ravel(), gf.cpu().numpy()]),
                np.concatenate([ogt.ravel(), ogp]), rel=tol, entry=tol)


def test_filter_improbable_observation():
    """A landmark seen far from where the belief has its mass: the sum falls
    by many powers of ten in one step and the filter goes on."""
    _say("filter improbable observation")
    from paper_1810_00204_amd.filter import FilterProblem
    prob, theta, phi, acts, obs = _set(30, 20, 1, 8, 6, False, seed=3)
    b0 = np.full(prob.S, 1e-25)
    b0[prob.occ != 0] = 0.0
    b0[np.flatnonzero(prob.occ == 0)[-1]] = 1.0
    prob.b0 = (b0 / b0.sum()).astype(np.float32)
    obs = obs % 16
    obs[0, 1] += 16   # landmark 1, near the top
    fp = FilterProblem(prob, acts, obs, ckpt_every=3)
    nll, gs, gf = fp.run(torch.as_tensor(theta), torch.as_tensor(phi))
    torch.cuda.synchronize()
    onll, ogt, ogp = oracle.filter_nll_grad(prob, theta, phi, acts, obs)
    assert onll[0] > 40
    np.testing.assert_allclose(nll.cpu().numpy(), onll, rtol=2e-5)
    _grad_close(np.concatenate([gs.cpu().numpy().ravel(), gf.cpu().numpy()]),
                np.concatenate([ogt.ravel(), ogp]))
