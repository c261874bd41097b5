"""GPU parity of the point-wise kernels at the edges of their tiles, through the fused call (LK^c and Conv_fuse)
against the CPU oracle; the bars are the fused call's (tests/test_gpu_fused.py)."""
import numpy as np
import pytest

from paper_2503_06671_amd import workloads as wk
from tests.test_gpu_fused import check_fused, pointwise_weights, residual_for, run_fused

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


@pytest.mark.parametrize("N", [1, 600])   # one and two pixels per lane
def test_values_that_have_no_three_bf16_terms(N):
    # fp32 storage: an infinite pixel gives an infinity of each weight's sign, one beyond the largest bf16 its
    # finite product, two infinities what their sum gives, in every output channel and nowhere else
    C, H, W, Ca = 12, 3, 7, 4
    wl = wk.make_random(950 + N, N, C, H, W, Ca, 3, dtype=F32, x_mean=0.3)
    w_fuse, b_fuse, _ = pointwise_weights(951, C, Ca)
    clean = run_fused(wl, w_fuse, b_fuse, None, residual_for(wl, 952))
    x = wl.x
    planted = [(0, Ca, 0, 0, np.inf), (N - 1, C - 1, 2, 6, -np.inf), (N // 2, Ca + 1, 1, 3, 3.4e38),
               (N // 2, Ca + 2, 1, 4, np.inf), (N // 2, Ca + 5, 1, 4, np.inf)]
    for n, c, y, xx, v in planted:
        x[n, c, y, xx] = v
    got = run_fused(wl, w_fuse, b_fuse, None, residual_for(wl, 952))
    touched = np.zeros((N, H, W), bool)
    for n, _, y, xx, _ in planted:
        touched[n, y, xx] = True
    assert np.array_equal(got[~np.broadcast_to(touched[:, None], got.shape)], clean[~np.broadcast_to(touched[:, None], got.shape)])
    for n, y, xx in np.argwhere(touched):
        big = x[n, Ca:, y, xx].astype(np.float64)
        with np.errstate(invalid="ignore"):
            want = (w_fuse[:, Ca:].astype(np.float64) * big).sum(1)   # beside these the other terms vanish
        have = got[n, :, y, xx].astype(np.float64)
        print(f"[case] N={N} pixel {n},{y},{xx}", flush=True)
        assert np.array_equal(np.isnan(have), np.isnan(want)) and np.array_equal(np.isinf(have), np.isinf(want))
        fin = np.isfinite(want)
        assert np.array_equal(have[~fin & ~np.isnan(want)], want[~fin & ~np.isnan(want)])
        assert np.allclose(have[fin], want[fin], rtol=1e-5, atol=0)
