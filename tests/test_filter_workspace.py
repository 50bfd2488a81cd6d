"""The filter's workspace stays within 512 MiB of stored beliefs, or what one
concurrent run per CU (256) takes for the bare cells, whichever is more: runs
that share a CU, and strips that go beyond the grid, must not take more.  Host
logic only; no kernel runs."""
import pytest

from paper_1810_00204_amd import binding as B
from paper_1810_00204_amd import workloads as wl
from tests.test_lib_host import FakeModel


@pytest.mark.parametrize("W,H,ntraj,T,k", [
    (24, 24, 4096, 2000, 10), (24, 24, 4096, 2000, 1), (24, 24, 64, 2000, 10), (10, 10, 4096, 2000, 10),
    (3, 2, 1000, 100000, 300), (64, 64, 2048, 200, 14), (33, 33, 700, 1000, 1000),
    (133, 133, 1024, 500, 22), (128, 128, 1024, 50, 10), (100, 40, 1, 1000, 30)])
def test_filter_workspace_is_bounded(W, H, ntraj, T, k):
    m = FakeModel(wl.make_small(seed=1, W=W, H=H))
    nb = B.qv_filter_workspace_bytes(m, ntraj, T, k)
    assert nb > 0
    run = ((T + k - 1) // k + k + 2) * W * H * 4 + (T + 1) * 4
    beside = W * H * 4 + 9 * 1024 + ntraj * 85 * 8 + 8 * 256
    assert nb <= max(512 << 20, min(ntraj, 256) * run) + beside
