"""Items of a batch's level by action below 512 (parent, band) pairs and by
parent from there on: the same queries in a batch on either side of the line
give the same trees, bit for bit, and the FP64 oracle's."""
import pytest

import oracle
from paper_1810_00204_amd import workloads as wl
from tests import parity
from tests.test_gpu_batch import SEED, _gpu_q, _same_tree, _say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("chunk", [1, 3])
def test_batch_items_on_both_sides_of_the_line(chunk):
    _say(f"batch items by action and by parent, {chunk} a visit")
    from paper_1810_00204_amd.planner import BatchPlanner
    # pairs at level 0 in bands of 256 cells: 5 + 10 + 4 per 32 x 32 query
    probs = [wl.make_paper(seed=81, W=33, H=35, D=2, n=3),
             wl.make_rect(seed=82, side=47, n_landmarks=9, D=2, n=3)]
    probs += [wl.make_small(seed=90 + q, W=32, H=32, D=2, n=3) for q in range(126)]
    Qs = [_gpu_q(p) for p in probs]
    trees = []
    for nq in (126, 128):   # 511 and 519 pairs
        bp = BatchPlanner(probs[:nq], Qs[:nq], n=3)
        bp.set_shape(256, chunk)
        for _ in range(2):
            acts, rq = bp.plan(SEED)
        trees.append(([bp.tree(q) for q in range(126)], acts[:126].clone(), rq[:126].clone()))
    (t1, a1, r1), (t2, a2, r2) = trees
    assert torch.equal(a1, a2) and torch.equal(r1, r2)
    for x, y in zip(t1, t2):
        _same_tree(x, y)
    for q in (0, 1, 2, 125):
        p = probs[q]
        res = oracle.plan(p, Qs[q].cpu().numpy().reshape(p.W * p.H, -1).astype("f8"), seed=SEED, qid=q)
        parity.compare_tree(p, t2[q], res["dump"], check_beliefs=False)
        assert parity.root_action_ok(int(a2[q]), res["rootQ"], res["action"])
