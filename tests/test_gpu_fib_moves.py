"""The FIB solve by the moves of its slip rows: all eight of every action, five
to seven, and some actions with all eight beside sparse ones; a single action,
which takes the blind bound's kernels; and more sweeps than one look at the
residuals covers.  Against the FP64 oracle's sweeps, with the tolerance of
test_gpu_fib_forms.py, and the two forms against each other bit for bit."""
import numpy as np
import pytest

import oracle
from paper_1810_00204_amd import binding as B
from tests.test_gpu_fib_forms import _problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _solve(prob, n, tol=0.0):
    m = B.DeviceModel(prob, "cuda")
    al = torch.empty(m.S * m.A, dtype=torch.float32, device="cuda")
    ws = torch.empty(B.qv_fib_workspace_bytes(m, n), dtype=torch.uint8, device="cuda")
    st, res, sw = B.qv_fib_iterate(m, tol, n, al, ws)
    assert st == 0
    return al.cpu().numpy(), res, sw


def _rows(prob, kind, seed):
    """Slip rows of the kind: `some` five to seven moves each, `mixed` the first
    action's row dense, the others as they are."""
    rng = np.random.default_rng([1810, seed])
    slip = prob.slip.astype(np.float64).copy()
    if kind == "some":
        for a in range(prob.A):
            off = rng.choice([0, 1, 2, 3, 5, 6, 7, 8], size=rng.integers(1, 4), replace=False)
            slip[a] = rng.dirichlet(np.ones(9))
            slip[a, off] = 0.0
    else:
        slip[0] = rng.dirichlet(np.ones(9))
    prob.slip = (slip / slip.sum(1, keepdims=True)).astype(np.float32)


def _check(prob, al, n):
    ref, _, osw = oracle.fib_iterate(prob, tol=0.0, max_sweeps=n)
    assert osw == n
    ref = np.asarray(ref).reshape(-1)
    bound = 40 * 2.0 ** -24 * np.abs(ref).max() * (1 - 0.95 ** n) / 0.05
    err = np.abs(al - ref).max()
    assert err <= bound, (err, bound)
    assert not al.reshape(prob.S, prob.A)[prob.occ != 0].any()


@pytest.mark.parametrize("kind", ["some", "mixed"])
@pytest.mark.parametrize("W,H,A,L", [(9, 8, 2, 2), (33, 21, 4, 5), (16, 13, 6, 4), (40, 30, 8, 30),
                                     (21, 22, 9, 12)])
def test_fib_moves_match_oracle(W, H, A, L, kind, monkeypatch):
    print(f"[case] fib {W}x{H} A{A} L{L} {kind} moves", flush=True)
    prob = _problem(W, H, A, L, False, True, 2)
    _rows(prob, kind, A)
    outs = []
    for form in ("QVTS_SWEEP_LAUNCHES", "QVTS_SWEEP_COOP"):
        monkeypatch.setenv(form, "1")
        outs.append(_solve(prob, 30)[0])
        monkeypatch.delenv(form)
    assert np.array_equal(*outs)
    _check(prob, outs[0], 30)


@pytest.mark.parametrize("W,H,L,dense", [(5, 4, 0, False), (19, 23, 9, True), (70, 66, 40, False)])
def test_fib_of_one_action_matches_oracle(W, H, L, dense):
    print(f"[case] fib {W}x{H} A1 L{L} dense {dense}", flush=True)
    prob = _problem(W, H, 1, L, dense, True, 3)
    _check(prob, _solve(prob, 30)[0], 30)


@pytest.mark.parametrize("W,H,A,dense", [(20, 20, 4, False), (31, 33, 8, True)])
def test_fib_beyond_one_look_at_the_residuals(W, H, A, dense, monkeypatch):
    """Per-sweep launches are looked at every 64 sweeps: 70 sweeps, and a
    tolerance that the solve meets between sweeps 64 and 128."""
    print(f"[case] fib {W}x{H} A{A}, past 64 sweeps", flush=True)
    prob = _problem(W, H, A, 3, dense, True, 4)
    res = {}
    for form in ("QVTS_SWEEP_LAUNCHES", "QVTS_SWEEP_COOP"):
        monkeypatch.setenv(form, "1")
        res[form] = [_solve(prob, 70), _solve(prob, 400, tol=1e-3)]
        monkeypatch.delenv(form)
    one, two = res.values()
    for (a, ra, sa), (b, rb, sb) in zip(one, two):
        assert np.array_equal(a, b) and ra == rb and sa == sb
    assert one[0][2] == 70 and 64 < one[1][2] < 128, one[1][2]
    _check(prob, one[0][0], 70)
