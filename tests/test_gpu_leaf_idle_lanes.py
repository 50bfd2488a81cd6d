"""The last level on maps whose first leaf band (8192 cells) has no free cell:
the sorted list's first positions are then never written, and the lanes
without a chunk must not take a cell from them.  The workspace is filled with
ones first, which read as the largest cell index.  Against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_1810_00204_amd import binding as B
from paper_1810_00204_amd import workloads as wl
from tests import parity
from tests.test_gpu_batch import SEED
from tests.test_gpu_plan import PATHS, _q32, _say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _top_blocked(W, H, A, L):
    """W x H, the first 8192 cells blocked, the rest with 15% walls."""
    rng = np.random.default_rng([1810, W, H, A])
    occ = wl.occ_exact_count(rng, W, H, 0.15)
    occ[:8192 // W * W] = 1
    free = rng.permutation(np.flatnonzero(occ == 0))
    goal = int(free[0])
    slip = {2: wl.slip_table_4, 4: wl.slip_table_4, 8: wl.slip_table_8}[A]()[:A]
    return wl.Problem(name="", W=W, H=H, occ=occ, slip=slip, flip=np.full(4, 0.1, np.float32),
                      lm_cell=np.sort(free[10:10 + L]).astype(np.int32), lm_p=0.8,
                      R=wl.reward_step_goal(occ, W, H, slip, goal), goal=goal, gamma=0.95,
                      b0=wl.belief_uniform_cells(W * H, free[1:6]), D=2, n=3, seed=7)


@pytest.mark.parametrize("path", list(PATHS))
@pytest.mark.parametrize("W,H,A,L", [(64, 200, 4, 0), (64, 140, 8, 9), (100, 130, 2, 0),
                                     (128, 200, 8, 0)])
def test_plan_with_a_blocked_first_band(W, H, A, L, path):
    _say(f"plan {W}x{H} A{A} L{L} path={path}, first band blocked")
    from paper_1810_00204_amd.planner import Planner
    prob = _top_blocked(W, H, A, L)
    Q32 = _q32(prob)
    pl = Planner(prob, flags=PATHS[path])
    pl.ws.fill_(255)
    act, _ = pl.plan(torch.as_tensor(Q32.reshape(-1)).cuda())
    g = pl.tree(beliefs=False)
    res = oracle.plan(prob, Q32)
    parity.compare_tree(prob, g, res["dump"], check_beliefs=False)
    assert parity.root_action_ok(int(act.item()), res["rootQ"], res["action"])


def test_batch_with_blocked_first_bands():
    _say("batch, first bands blocked")
    from paper_1810_00204_amd.planner import BatchPlanner
    probs = [_top_blocked(64, 200, 4, 0), _top_blocked(64, 140, 8, 9), _top_blocked(100, 130, 2, 0)]
    Qs = [_q32(p) for p in probs]
    bp = BatchPlanner(probs, Qs, n=3)
    bp.ws.fill_(255)
    acts, _ = bp.plan(SEED)
    acts = acts.cpu().numpy()
    for q, p in enumerate(probs):
        res = oracle.plan(p, Qs[q].astype(np.float64), seed=SEED, qid=q)
        parity.compare_tree(p, bp.tree(q), res["dump"], check_beliefs=False)
        assert parity.root_action_ok(int(acts[q]), res["rootQ"], res["action"])
