"""The children's bounds over table widths on both sides of the staged rows'
limit (12 columns), cell counts below a wavefront, off its multiples and above
a workgroup, and more samples than one group of a climb's reads, against the
FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_1810_00204_amd import workloads as wl
from tests.test_gpu_search import _compare, _say, _tables

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("W,H,cols,n", [(6, 5, 4, 2), (13, 9, 1, 3), (20, 12, 12, 5),
                                        (20, 12, 13, 2), (40, 33, 9, 3), (9, 7, 17, 4)])
def test_search_table_widths_match_oracle(W, H, cols, n):
    from paper_1810_00204_amd.planner import SearchPlanner
    _say(f"search {W}x{H}, {cols} lower columns, {n} samples")
    prob = wl.make_small(seed=80 + W, W=W, H=H, D=2, n=n)
    U32, L32 = _tables(prob)
    # any number of lower-bound columns: the blind policies' own, each again
    # lowered by a little
    L32 = np.stack([L32[:, c % L32.shape[1]] - np.float32(0.01 * (c // L32.shape[1]))
                    for c in range(cols)], axis=1).astype(np.float32)
    steps = 16
    sp = SearchPlanner(prob, U32, L32, max_nodes=1 + steps * prob.A * n)
    sp.init()
    sp.expand(steps, seed=prob.seed, query_id=5)
    sp.result()
    t = oracle.search(prob, U32, L32, steps, seed=prob.seed, qid=5)
    assert _compare(prob, sp.records(), t) > 0
