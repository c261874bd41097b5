"""GPU parity of the point-wise kernels at the edges of their tiles, through the fused call (LK^c and Conv_fuse)
against the CPU oracle; the bars are the fused call's (tests/test_gpu_fused.py)."""
import pytest

from paper_2503_06671_amd import workloads as wk
from tests.test_gpu_fused import check_fused, pointwise_weights, residual_for

pytestmark = pytest.mark.gpu

F32, BF16 = wk.F32, wk.BF16


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("N,C,H,W,Ca", [
    (1, 16, 1, 31, 5),      # a chunk of 16 channels that ends one tensor and starts the other; one pixel short of a wavefront's 32
    (1, 17, 1, 33, 16),     # one channel and one pixel more
    (1, 33, 8, 16, 16),     # 33 output channels: a second row block of one row; 128 pixels
    (1, 64, 3, 43, 24),     # tensors that meet in the middle of a chunk (24 = 16 + 8); 129 pixels
    (1, 65, 5, 7, 12),      # a second group of output channels
    (1, 240, 4, 9, 48),     # the widest
    (600, 20, 3, 5, 7),     # two pixels per lane: odd planes, the last lane takes its neighbour's last pixel again
    (300, 40, 2, 129, 16),  # two pixels per lane, two pixels into a second tile
    (520, 6, 1, 1, 3),      # planes of a single pixel, however many: one pixel per lane
])
def test_tile_edges(oracle, dtype, N, C, H, W, Ca):
    wl = wk.make_random(900 + C + H, N, C, H, W, Ca, 3, dtype=dtype, x_mean=0.3)
    w_fuse, b_fuse, lkc = pointwise_weights(901 + C, C, Ca)
    check_fused(wl, oracle, w_fuse, b_fuse, lkc, residual_for(wl, 902), what=f"{N}x{C}x{H}x{W} Ca={Ca}")
