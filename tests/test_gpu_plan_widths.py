"""Plans on grids whose width lies at the edges of a wavefront's row pieces
(several rows a piece up to 32 columns, one piece a row to 64, several beyond;
partial pieces, bands cut at the grid's edges), with a goal and landmarks,
against the FP64 oracle."""
import pytest

from paper_1810_00204_amd import binding as B
from paper_1810_00204_amd import workloads as wl
from tests.test_gpu_plan import PATHS, _check, _q32, _say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("path", list(PATHS))
@pytest.mark.parametrize("W,H", [(2, 40), (3, 5), (31, 33), (32, 31), (33, 40), (63, 20),
                                 (64, 64), (65, 17), (128, 9), (129, 30), (260, 40)])
def test_plan_widths_match_oracle(W, H, path):
    _say(f"plan {W}x{H} path={path}")
    prob = wl.make_small(seed=60 + W, W=W, H=H, D=2, n=3)
    _check(prob, _q32(prob), flags=PATHS[path], beliefs=False)


@pytest.mark.parametrize("side", [32, 33, 96])
def test_plan_sides_with_landmarks_match_oracle(side):
    _say(f"plan {side}x{side} with landmarks")
    prob = wl.make_rect(seed=70 + side, side=side, n_landmarks=24, D=2, n=3)
    _check(prob, _q32(prob), flags=B.QV_PLAN_TILED, beliefs=False)
