"""Items of the batch's launches: per-parent items over all actions and (for
bands of more than 2048 cells) items per action, a last level of 9 actions,
and levels with many more items than resident workgroups, against the FP64
oracle; and the same tree bit for bit however many items a visit takes."""
import gc

import numpy as np
import pytest

import oracle
from paper_1810_00204_amd import binding as B
from paper_1810_00204_amd import workloads as wl
from tests import parity
from tests.test_gpu_batch import SEED, _gpu_q, _same_tree, _say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _give_back():
    """Large workspaces go back to the device: later tests read slots that a
    plan leaves unwritten, and the -1 records here are NaNs as floats."""
    yield
    gc.collect()
    torch.cuda.empty_cache()


def _check(probs, bp, Qs, acts, picks):
    for q in picks:
        p = probs[q]
        p.n = 3
        Q = Qs[q].cpu().numpy().reshape(p.W * p.H, -1).astype(np.float64)
        res = oracle.plan(p, Q, seed=SEED, qid=q)
        parity.compare_tree(p, bp.tree(q), res["dump"], check_beliefs=False)
        assert parity.root_action_ok(int(acts[q]), res["rootQ"], res["action"])


@pytest.mark.parametrize("tile", [256, 2048, 4096])
def test_batch_items_per_parent_and_per_action(tile):
    """Bands of 2048 cells and less take per-parent items, above that (70 x 50
    and 64 x 64 at 4096) items per action."""
    _say(f"batch items, {tile} cells per band")
    from paper_1810_00204_amd.planner import BatchPlanner
    probs = [wl.make_paper(seed=41, W=70, H=50, D=2, n=3),
             wl.make_small(seed=42, W=64, H=64, D=3, n=3),
             wl.make_rect(seed=43, side=47, n_landmarks=9, D=2, n=3),
             wl.make_small(seed=44, W=33, H=5, D=1, n=3)]
    Qs = [_gpu_q(p) for p in probs]
    bp = BatchPlanner(probs, Qs, n=3)
    bp.set_shape(tile, 1)
    acts, _ = bp.plan(SEED)
    _check(probs, bp, Qs, acts.cpu().numpy(), range(len(probs)))


@pytest.mark.parametrize("chunk", [2, 4])
def test_batch_many_items_per_workgroup(chunk):
    """24 queries of 48 x 48 in bands of 5 rows: tens of thousands of items
    per launch, so every workgroup takes many times."""
    _say(f"batch items, {chunk} a visit")
    from paper_1810_00204_amd.planner import BatchPlanner
    probs = [wl.make_small(seed=50 + q, W=48, H=48, D=3, n=3) for q in range(24)]
    Qs = [_gpu_q(p) for p in probs]
    one = BatchPlanner(probs, Qs, n=3)
    one.set_shape(256, 1)
    a1, r1 = one.plan(SEED)
    bp = BatchPlanner(probs, Qs, n=3)
    bp.set_shape(256, chunk)
    for _ in range(3):
        acts, rq = bp.plan(SEED)
        assert torch.equal(acts, a1) and torch.equal(rq, r1)
    for q in range(24):
        _same_tree(bp.tree(q), one.tree(q))
    _check(probs, bp, Qs, acts.cpu().numpy(), (0, 23))
