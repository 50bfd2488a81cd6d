"""Slots that a plan never writes (values of absent nodes): a planner's tree
holds zeros there, not what the allocator's memory held before, so that two
reads of it compare equal."""
import numpy as np
import pytest

from paper_1810_00204_amd import binding as B
from paper_1810_00204_amd import workloads as wl
from tests.test_gpu_plan import PATHS, _q32, _say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("path", list(PATHS))
def test_unwritten_slots_do_not_depend_on_old_memory(path):
    _say(f"plan, unwritten slots, path={path}")
    from paper_1810_00204_amd.planner import Planner
    prob = wl.make_rect(seed=12, side=40, D=3, n=3)
    Qd = torch.as_tensor(_q32(prob).reshape(-1)).cuda()
    trees = []
    for fill in (0xFF, 0x11):
        m = B.DeviceModel(prob, "cuda")
        nb = B.qv_plan_workspace_bytes(m, prob.D, prob.n, PATHS[path])
        old = torch.empty(nb, dtype=torch.uint8, device="cuda")
        old.fill_(fill)   # what the planner's workspace is cut from next
        del old, m
        pl = Planner(prob, flags=PATHS[path])
        pl.plan(Qd)
        trees.append(pl.tree(beliefs=True))
        del pl
    t1, t2 = trees
    absent = t1["valid"] == 0
    assert absent.any()
    for k in ("valid", "z", "count", "pz", "value", "qvalue", "reward"):
        assert np.array_equal(t1[k], t2[k]), k
    for d in t1["beliefs"]:
        assert np.array_equal(t1["beliefs"][d], t2["beliefs"][d])
