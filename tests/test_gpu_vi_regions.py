"""Value iteration in regions: grids of one region and just beyond, several
regions with remainders on both sides, every column count the kernel is built
for, few and all moves, a goal or none, and rules that fire at any sweep of a
launch.

Single-sweep launches and several sweeps per launch must agree bit for bit
(same arithmetic per cell).  Against the FP64 oracle's sweeps: a backup has at
most 11 roundings of 2^-24 relative to the largest |V| (nine products, gamma,
R), damped by gamma from sweep to sweep."""
import numpy as np
import pytest

import oracle
from paper_1810_00204_amd import binding as B
from tests.test_gpu_fib_forms import _problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _vi(prob, tol, most):
    m = B.DeviceModel(prob, "cuda")
    Q = torch.full((m.S * m.A,), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(B.qv_vi_workspace_bytes(m, most), dtype=torch.uint8, device="cuda")
    st, res, sw = B.qv_value_iterate(m, tol, most, Q, ws)
    assert st == 0
    return Q.cpu().numpy(), res, sw


@pytest.mark.parametrize("W,H,A,dense,goal", [
    (1, 1, 1, False, False), (20, 20, 4, False, True), (48, 50, 8, False, True),
    (49, 50, 8, True, True), (48, 51, 9, False, False), (33, 69, 2, True, False),
    (97, 103, 5, True, True), (130, 36, 3, False, False), (64, 64, 9, True, True)])
def test_value_iteration_regions(W, H, A, dense, goal, monkeypatch):
    print(f"[case] vi {W}x{H} A{A} dense {dense} goal {goal}", flush=True)
    prob = _problem(W, H, A, 0, dense, goal and W > 1, 2)
    for tol, most in ((0.0, 1), (0.0, 7), (0.0, 70), (1e-2, 500), (3e-3, 500), (1e-3, 500),
                      (3e-4, 500), (1e-5, 500)):
        monkeypatch.delenv("QVTS_SWEEP_LAUNCHES", raising=False)
        Q, res, sw = _vi(prob, tol, most)
        monkeypatch.setenv("QVTS_SWEEP_LAUNCHES", "1")
        Q1, res1, sw1 = _vi(prob, tol, most)
        assert (res, sw) == (res1, sw1)
        assert np.array_equal(Q, Q1)
        if tol == 0.0:
            ref, _, osw = oracle.value_iterate(prob, tol=0.0, max_sweeps=most)
            if osw != sw:   # (an exact fixed point on the smallest grids)
                continue
            ref = np.asarray(ref).reshape(-1)
            bound = 11 * 2.0 ** -24 * (np.abs(ref).max() + 2) * (1 - 0.95 ** sw) / 0.05
            assert np.abs(Q - ref).max() <= bound
