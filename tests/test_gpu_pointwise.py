"""GPU parity of the point-wise kernels at the edges of their tiles, through the fused call (LK^c and Conv_fuse)
against the CPU oracle; the bars are the fused call's (tests/test_gpu_fused.py)."""
import numpy as np
import pytest
import torch

from paper_2503_06671_amd import binding, workloads as wk
from tests.test_gpu_ffn import check_ffn
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


# Channels in whole runs of sixteen: one to eight stages, the last one half full or full, both tensors' border inside a stage
# and between two, with and without the residual that takes an input buffer over; many images: two pixels per lane (from
# 512 groups of up to 64 output channels of an image on).
@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("N,C,Ca", [(1, 16, 16), (1, 32, 16), (2, 48, 16), (1, 64, 32), (1, 80, 48), (2, 96, 32), (1, 112, 16),
                                    (1, 128, 64), (1, 240, 48), (600, 32, 16), (600, 48, 32), (600, 64, 16), (300, 80, 16)])
def test_stages_of_whole_runs(oracle, dtype, N, C, Ca):
    wl = wk.make_random(960 + C, N, C, 3, 45, Ca, 3, dtype=dtype, x_mean=0.3)
    w_fuse, b_fuse, lkc = pointwise_weights(961 + C, C, Ca)
    check_fused(wl, oracle, w_fuse, b_fuse, lkc, residual_for(wl, 962), what=f"{N}x{C} Ca={Ca} residual")
    check_fused(wl, oracle, w_fuse, None, lkc, what=f"{N}x{C} Ca={Ca}")


# The same widths on maps large enough for two pixels per lane (planes of one tile: two images to a compute unit), whatever
# becomes of the sums: nothing, a residual, a GELU (a hidden layer beyond 128 channels takes the layers' own launches).
@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("C,Ca", [(16, 0), (16, 16), (32, 0), (32, 16), (32, 32), (48, 16), (64, 32), (80, 16)])
def test_whole_runs_two_pixels_per_lane(oracle, dtype, C, Ca):
    N = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    wl = wk.make_random(970 + C, N, C, 3, 15, Ca, 3, dtype=dtype, x_mean=0.3)
    w_fuse, b_fuse, lkc = pointwise_weights(971 + C, C, Ca)
    for residual in (None, residual_for(wl, 972)):
        check_fused(wl, oracle, w_fuse, b_fuse, lkc if Ca else None, residual, what=f"{N}x{C} Ca={Ca}")
    check_ffn(oracle, 973, N, C, 3, 15, 160, dtype)


@pytest.mark.parametrize("N,C", [(1, 20), (1, 40), (1, 64), (1, 96), (600, 24), (600, 32), (600, 64), (600, 70)])  # one to three stages of channels, one and two row blocks and pixels per lane
@pytest.mark.parametrize("Ca", [8, 16])   # 16: the kernels for whole runs, where C is one too
def test_residual_is_rounded_once(N, C, Ca):
    # fp32 storage: the residual is added to the finished sums, so that one far larger than they are costs them no
    # more than the one rounding of that addition
    H, W = 3, 15
    wl = wk.make_random(930 + C, N, C, H, W, Ca, 3, dtype=F32, x_mean=0.3)
    w_fuse, b_fuse, _ = pointwise_weights(931, C, Ca)
    res = 100 * residual_for(wl, 932)
    print(f"[case] residual added once N={N} C={C}", flush=True)
    assert np.array_equal(run_fused(wl, w_fuse, b_fuse, None, res), run_fused(wl, w_fuse, b_fuse) + res)


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


@pytest.mark.parametrize("what", ["x", "last channel", "w1", "w2", "one weight"])
def test_nan_costs_no_more_than_a_few_ordinary_calls(what):
    # fp32 storage: an element that is NaN because a value or weight of it is must not be summed again
    # (three launches, 16 x 96 -> 192 -> 96 channels of 64 x 64: it took 55 to 80 times an ordinary call so, and takes
    # about twice as long with the rows and pixels found first; the bar is five times)
    N, C, H, W, Ch = 16, 96, 64, 64, 192
    g = torch.Generator(device="cuda")
    g.manual_seed(960)
    r = lambda *s: torch.randn(s, generator=g, device="cuda") * 0.1
    x, w1, k, w2 = r(N, C, H, W), r(Ch, C), r(Ch, 3, 3), r(C, Ch)
    ws, out = binding.new_convffn_workspace(N, Ch, H, W, torch.float32), torch.empty_like(x)

    def us():
        times = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                binding.convffn_forward(x, w1, k, w2, ws, out=out)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 200.0)
        return sorted(times)[3]

    print(f"[case] cost of NaN: {what}", flush=True)
    ordinary = us()
    assert torch.isfinite(out).all()
    {"x": x, "last channel": x[:, -1], "w1": w1, "w2": w2, "one weight": w1[7, -1]}[what].fill_(float("nan"))
    with_nan = us()
    print(f"{what}: {ordinary:.1f} us, with NaN {with_nan:.1f} us", flush=True)
    assert torch.isnan(out).all()
    assert with_nan <= 5 * ordinary


@pytest.mark.parametrize("N,C", [(1, 32), (1, 64), (600, 64), (1, 96), (600, 80), (2, 192), (130, 112)])
def test_values_and_weights_of_any_size(N, C):
    # fp32 storage: a common factor of the values, of a row of weights, or of the channels of one stage beside another's
    # (2^12 here: a later stage's values a thousand times the first's, the other way round, and pixels without any) leaves
    # the error against float64 where fp32 sums have it.  K products and sums, each within 2^-24 of terms whose squares add
    # up: sqrt(2 K) 2^-24 of the result, and the weights' terms and the dropped product within 2^-23.
    H, W = 3, 45
    rng = np.random.default_rng(940 + C)
    w0, x0 = rng.standard_normal((C, C)) / np.sqrt(C), rng.standard_normal((N, C, H, W)) + 0.3
    bound = (np.sqrt(2 * C) / 2 + 1) * 2.0 ** -23
    first, second = np.ones((C, 1, 1)), np.ones((C, 1, 1))
    first[:C // 2], second[C // 2:] = 2.0 ** -12, 2.0 ** -12
    some = np.ones((1, H, W))
    some[:, :, W // 2:] = 0.0
    rows = 2.0 ** rng.integers(-60, 60, (C, 1))
    late = (np.arange(C) >= (32 if C > 32 else 0)).astype(float)[:, None]   # no weight and no value in the first stage
    for what, xs, ws in (("2^-30", 2.0 ** -30, 1.0), ("2^30", 2.0 ** 30, 1.0), ("2^-100 x 2^60", 2.0 ** -100, 2.0 ** 60), ("rows", 1.0, rows),
                         ("small first", first, 1.0), ("small last", second, 1.0), ("both", first * 2.0 ** -20, rows), ("zeros", some * 2.0 ** 14, 1.0),
                         ("late", late[:, :, None] * 2.0 ** -24, late.T * 2.0 ** -20)):
        x, w = (x0 * xs).astype(np.float32), (w0 * ws).astype(np.float32)
        wl = wk.make_random(941, N, C, H, W, 0, 3, dtype=F32)
        wl.x[...] = x
        print(f"[case] {what} N={N} C={C}", flush=True)
        got = run_fused(wl, w).astype(np.float64)
        want = np.einsum("mk,nkp->nmp", w.astype(np.float64), x.reshape(N, C, -1).astype(np.float64), optimize=True).reshape(got.shape)
        scale = np.sqrt((want ** 2).mean(axis=(0, 2, 3), keepdims=True))   # rows of W differ in size, and so do their results
        err = np.sqrt((((got - want) / scale) ** 2).mean())
        assert err <= bound, (what, err, bound)


def sum_bound(w, x):
    # |error| of sums of K fp32 products, each product and each addition rounded at most twice: K + 4 units of 2^-23 of the
    # sum of magnitudes, whatever their order
    return (w.shape[1] + 4) * 2.0 ** -23 * np.einsum("mk,nkp->nmp", np.abs(w).astype(np.float64), np.abs(x).astype(np.float64), optimize=True)


@pytest.mark.parametrize("N,C", [(1, 12), (1, 64), (1, 96), (600, 64), (2, 192), (130, 112)])   # one and two pixels a lane, two to seven stages
def test_a_pixel_depends_on_itself_alone(N, C):
    # fp32 storage: finite values of any size, in any channel, cost their own pixel's sums no more than fp32 arithmetic
    # does, and the other pixels nothing; infinities likewise.  (32784 and 40016 are values whose rest behind the
    # nearest fp16 is 16.)
    H, W = 3, 45
    w, _, _ = pointwise_weights(981 + C, C, 0)
    wl = wk.make_random(980 + C, N, C, H, W, 0, 3, dtype=F32, x_mean=0.3)
    clean = run_fused(wl, w)
    planted = [(C - 1, 0, 0, 32784.0), (C // 2 + 4, 0, 7, -40016.0), (C - 2, 0, 40, 1e5), (0, 1, 3, 1e8), (C - 1, 1, 30, -1e10), (C // 2, 2, 2, 1e12),
               (1, 2, 20, 1e30), (C - 3, 2, 33, np.inf)]
    touched = np.zeros((N, H, W), bool)
    for i, (c, y, xx, v) in enumerate(planted):
        wl.x[i % N, c, y, xx] = v
        touched[i % N, y, xx] = True
    print(f"[case] large pixels N={N} C={C}", flush=True)
    got = run_fused(wl, w)
    other = np.broadcast_to(~touched[:, None], got.shape)
    assert np.array_equal(got[other], clean[other])
    x = wl.x.reshape(N, C, -1)
    with np.errstate(invalid="ignore"):
        want = np.einsum("mk,nkp->nmp", w.astype(np.float64), x.astype(np.float64), optimize=True).reshape(got.shape)
        bound = sum_bound(w, x).reshape(got.shape)
    assert np.array_equal(np.isfinite(got), np.isfinite(want))
    fin = np.isfinite(want)
    assert (np.abs(got[fin].astype(np.float64) - want[fin]) <= bound[fin]).all()


@pytest.mark.parametrize("N,C", [(1, 64), (1, 96), (600, 64), (2, 192), (130, 112)])
def test_rows_and_pixels_of_any_range(N, C):
    # fp32 storage: weights behind the first 32 far larger or smaller than those, channels likewise, each sum within fp32's own
    # bound of magnitudes; a weight of one alone moves the values as they are.
    H, W = 3, 45
    wl = wk.make_random(990 + C, N, C, H, W, 0, 3, dtype=F32, x_mean=0.3)
    x0 = wl.x.copy()
    w0, _, _ = pointwise_weights(991 + C, C, 0)
    late = np.where(np.arange(C) < 32, 1.0, 0.0)
    for what, xs, ws in (("late weights 2^15", 1.0, 2.0 ** -15 * late + (1 - late)), ("late weights 2^20", 1.0, 2.0 ** -20 * late + (1 - late)),
                         ("late weights 2^-40", 1.0, late + 2.0 ** -40 * (1 - late)), ("late channels 2^40", 2.0 ** -40 * late + (1 - late), 1.0),
                         ("late channels 2^-40", late + 2.0 ** -40 * (1 - late), late * 2.0 ** -40 + (1 - late))):
        print(f"[case] {what} N={N} C={C}", flush=True)
        w = (w0 * np.asarray(ws)).astype(np.float32)
        wl.x[...] = (x0 * np.asarray(xs).reshape(-1, *([1, 1] if np.ndim(xs) else []))).astype(np.float32)
        got = run_fused(wl, w).astype(np.float64)
        x = wl.x.reshape(N, C, -1)
        want = np.einsum("mk,nkp->nmp", w.astype(np.float64), x.astype(np.float64), optimize=True).reshape(got.shape)
        assert (np.abs(got - want) <= sum_bound(w, x).reshape(got.shape)).all(), what
    wl.x[...] = x0 * 2.0 ** np.random.default_rng(992).integers(-60, 60, x0.shape)
    assert np.array_equal(run_fused(wl, np.eye(C, dtype=np.float32)), wl.x)
