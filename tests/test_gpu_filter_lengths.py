"""The filter kernel at strip lengths 4, 6 and 8, plain and with landmarks and
a goal, along either side of the grid, and on narrow grids, whose bands have
wider rows.  Against the FP64 oracle, with the other filter sets' tolerances
(test_gpu_filter_adjoint.py)."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_filter_adjoint import _grad_close, _say
from tests.test_gpu_filter_strips import _set

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L,goal", [(0, False), (6, True)])
@pytest.mark.parametrize("W,H", [(20, 30), (30, 20),       # strips of 4
                                 (35, 33), (33, 35), (22, 48),   # of 6
                                 (52, 67), (67, 52),       # of 8
                                 (30, 60), (1000, 2), (2, 1000),   # of 8, wider rows
                                 (14, 512), (6, 600), (2000, 2)])   # of 16, wider rows
def test_filter_lengths_match_oracle(W, H, L, goal):
    _say(f"filter {W}x{H} L{L} goal {goal}")
    from paper_1810_00204_amd.filter import FilterProblem
    prob, theta, phi, acts, obs = _set(W, H, 3, 9, L, goal, seed=5)
    fp = FilterProblem(prob, acts, obs, ckpt_every=4)
    nll, gs, gf = fp.run(torch.as_tensor(theta), torch.as_tensor(phi))
    only, _, _ = fp.run(torch.as_tensor(theta), torch.as_tensor(phi), grad=False)
    torch.cuda.synchronize()
    onll, ogt, ogp = oracle.filter_nll_grad(prob, theta, phi, acts, obs)
    np.testing.assert_allclose(nll.cpu().numpy(), onll, rtol=2e-5)
    assert torch.equal(nll, only)
    _grad_close(np.concatenate([gs.cpu().numpy().ravel(), gf.cpu().numpy()]),
                np.concatenate([ogt.ravel(), ogp]))
