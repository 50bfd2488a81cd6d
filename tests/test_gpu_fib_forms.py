"""The FIB sweep over its forms: every column count it is built for, action
counts below it, slip rows with few and with all moves, landmarks and a goal,
one-launch and per-sweep, a remainder of the 64-cell groups, fewer than 64
free cells, and a reward table that is not 16-byte aligned, against the FP64
oracle's sweeps.

Tolerance: a sweep forms, per cell and action, at most 16 sums of nine
products with a likelihood of four factors, their sum, the landmark terms and
one product with gamma: at most 40 roundings of 2^-24 relative to the largest
|alpha|, damped by gamma from sweep to sweep."""
import numpy as np
import pytest

import oracle
from paper_1810_00204_amd import binding as B
from paper_1810_00204_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _problem(W, H, A, L, dense, goal, seed):
    rng = np.random.default_rng([1810, W, H, A, seed])
    occ = wl.occ_exact_count(rng, W, H, 0.25)
    free = np.flatnonzero(occ == 0)
    if dense:
        slip = rng.dirichlet(np.ones(9), A)
    else:
        slip = {4: wl.slip_table_4, 8: wl.slip_table_8, 9: wl.slip_table_9}[
            4 if A <= 4 else 8 if A <= 8 else 9]()[:A].astype(np.float64)
    slip = (slip / slip.sum(1, keepdims=True)).astype(np.float32)
    g = int(free[3]) if goal else -1
    R = rng.uniform(-2, 1, (W * H, A)).astype(np.float32)
    R[occ != 0] = 0
    lm = rng.permutation(free[free != g])[:L].astype(np.int32)
    return wl.Problem(name="", W=W, H=H, occ=occ, slip=slip,
                      flip=np.array([0.1, 0.2, 0.05, 0.15], np.float32), lm_cell=lm, lm_p=0.8, R=R,
                      goal=g, gamma=0.95, b0=wl.belief_uniform_cells(W * H, free))


@pytest.mark.parametrize("launches", [False, True])
@pytest.mark.parametrize("W,H,A,L,dense,goal", [
    (5, 4, 1, 0, False, False), (9, 8, 2, 2, True, True), (17, 15, 3, 0, True, False),
    (33, 21, 4, 5, False, True), (20, 20, 4, 0, True, False), (16, 13, 5, 4, True, True),
    (23, 19, 7, 0, False, False), (40, 30, 8, 30, False, True), (31, 33, 8, 9, True, False),
    (100, 40, 9, 0, False, False), (21, 22, 9, 12, True, True)])
def test_fib_forms_match_oracle(W, H, A, L, dense, goal, launches, monkeypatch):
    print(f"[case] fib {W}x{H} A{A} L{L} dense {dense} launches {launches}", flush=True)
    monkeypatch.setenv("QVTS_SWEEP_LAUNCHES" if launches else "QVTS_SWEEP_COOP", "1")
    prob = _problem(W, H, A, L, dense, goal, 1)
    m = B.DeviceModel(prob, "cuda")
    if dense:   # the reward table one float off its alignment
        R = torch.empty(m.S * A + 1, dtype=torch.float32, device="cuda")
        R[1:].copy_(torch.as_tensor(prob.R.reshape(-1)))
        m.c.R = R.data_ptr() + 4
    n = 40
    al = torch.empty(m.S * A, dtype=torch.float32, device="cuda")
    ws = torch.empty(B.qv_fib_workspace_bytes(m, n), dtype=torch.uint8, device="cuda")
    st, res, sw = B.qv_fib_iterate(m, 0.0, n, al, ws)
    assert st == 0 and sw == n
    ref, _, osw = oracle.fib_iterate(prob, tol=0.0, max_sweeps=n)
    assert osw == n
    ref = np.asarray(ref).reshape(-1)
    bound = 40 * 2.0 ** -24 * np.abs(ref).max() * (1 - 0.95 ** n) / 0.05
    err = np.abs(al.cpu().numpy() - ref).max()
    assert err <= bound, (err, bound)
    assert not al.cpu().numpy().reshape(m.S, A)[prob.occ != 0].any()
