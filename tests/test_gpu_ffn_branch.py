"""GPU parity of ConvFFN's depth-wise branch as a launch of its own at the edges of its strips, and of the one-launch
kernels on small images (bands of one to three rows), through the whole network against the CPU oracle; the bars are tests/test_gpu_ffn.py's."""
import numpy as np
import pytest

from paper_2503_06671_amd import workloads as wk
from tests.test_gpu_ffn import check_ffn, run_ffn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [wk.F32, wk.BF16])
@pytest.mark.parametrize("N,C,H,W,Ch", [
    (2, 5, 6, 3, 7),     # rows shorter than a 16-byte piece of either type
    (1, 5, 4, 4, 7),     # exactly a piece of fp32, half a piece of bf16; a strip that ends with the image
    (1, 5, 5, 7, 7),     # the last piece overlaps all but three elements of the one before; one row in the last strip
    (1, 5, 7, 8, 7),     # exactly a piece of bf16
    (2, 5, 8, 9, 7),     # one element more
    (1, 5, 3, 17, 7),    # two pieces and one element; fewer rows than a strip
    (3, 6, 9, 31, 10),   # odd planes: no piece is aligned, batches start anywhere
])
def test_strip_edges(oracle, dtype, N, C, H, W, Ch):
    check_ffn(oracle, 300 + H * W, N, C, H, W, Ch, dtype)


@pytest.mark.parametrize("dtype", [wk.F32, wk.BF16])
@pytest.mark.parametrize("N,C,H,W,Ch", [
    (1, 64, 1, 15, 128),    # one row, exactly half a strip
    (1, 64, 5, 14, 128),    # less than half a strip: three launches
    (2, 64, 64, 31, 128),   # bands of one row; a strip one column wide
    (3, 64, 83, 61, 128),   # bands of two rows, the last of one
    (1, 64, 134, 240, 128),   # bands of three rows, the last of two
    (1, 62, 11, 30, 100),   # just wide enough for the kernel's channels (62 x 100 of 64 x 96)
    (1, 61, 11, 30, 100),   # just not: three launches
])
def test_small_images(oracle, dtype, N, C, H, W, Ch):
    check_ffn(oracle, 400 + H * W, N, C, H, W, Ch, dtype)


@pytest.mark.parametrize("N,C,H,W,Ch", [
    (1, 64, 9, 31, 128),   # bands of one row
    (16, 6, 37, 100, 10),  # more bands and strips
])
def test_output_bias_is_rounded_once(N, C, H, W, Ch):
    # one launch, fp32 storage: b2 is added to the finished sums, so that one far larger than they are costs them no
    # more than that addition
    x = np.random.default_rng(480 + N + C).standard_normal((N, C, H, W)).astype(np.float32)
    p = wk.make_ffn_params(481 + C, C, Ch)
    b2 = 1000 * p["b2"]
    print(f"[case] output bias added once {N}x{C}x{H}x{W} Ch={Ch}", flush=True)
    assert np.array_equal(run_ffn(x, wk.F32, dict(p, b2=b2)), run_ffn(x, wk.F32, dict(p, b2=None)) + b2[:, None, None])


@pytest.mark.parametrize("what", ["values", "weight"])
@pytest.mark.parametrize("N,C,H,W,Ch", [
    (1, 64, 9, 31, 128),   # one launch, bands of one row
    (16, 6, 37, 100, 10),  # one launch, more bands and strips; channels that do not exist beside those that do
    (1, 6, 37, 100, 10),   # three launches
])
def test_values_that_have_no_three_bf16_terms(oracle, what, N, C, H, W, Ch):
    # fp32 storage: infinities, and finite inputs, hidden values and weights beyond the largest bf16, give what fp32
    # arithmetic gives, the same by either path.  Everything is positive, so no answer hangs on the order of a sum
    # (sums of positive terms: 1e-5 elementwise), and small enough that none overflows; gelu(-inf) is NaN
    rng = np.random.default_rng(500 + N + C)

    def pos(*shape, scale):
        return (rng.uniform(0.5, 1.0, shape) * scale).astype(np.float32)

    x = pos(N, C, H, W, scale=1.0)
    p = {"w1": pos(Ch, C, scale=0.5 / C), "b1": pos(Ch, scale=0.1), "k": pos(Ch, 3, 3, scale=0.1), "bk": pos(Ch, scale=0.1),
         "w2": pos(C, Ch, scale=0.2 / Ch), "b2": pos(C, scale=0.1)}
    p["w1"][1] = 1e-20
    if what == "values":
        p["w1"][1, 0] = 1    # hidden channel 1 is channel 0 of x, and so is V there (beside those the rest vanishes)
        p["k"][1], p["bk"][1] = 1e-20, 0
        for n, c, y, xx, v in [(0, 0, 0, 0, 3.4e38), (0, 0, 4, 15, 3.4e38), (0, 2, 4, 29, np.inf), (N - 1, C - 1, H - 1, W - 1, 3.4e38),
                               (N - 1, C - 1, H - 1, 3, np.inf), (N // 2, 1, 2, 20, -np.inf), (N // 2, 3, 7, 10, np.nan)]:
            x[n, c, y, xx] = v
    else:
        p["b1"][1], p["k"][1], p["bk"][1] = 0, 1e-20, 1e-3   # V is gelu(0.001) all over hidden channel 1
        p["w2"][C - 1, 1] = 3.4e38
        p["w1"][2, 1] = 3.4e38
        x[:, 1] *= np.float32(1e-3)
    print(f"[case] no three terms: {what} {N}x{C}x{H}x{W} Ch={Ch}", flush=True)
    got = run_ffn(x, wk.F32, p).astype(np.float64)
    with np.errstate(invalid="ignore", over="ignore"):
        ref = oracle.convffn_forward(x, p["w1"], p["k"], p["w2"], wk.F32, b1=p["b1"], bk=p["bk"], b2=p["b2"])
    if what == "values":
        assert np.isnan(ref).any() and np.isposinf(ref).any() and (ref[np.isfinite(ref)] > 1e35).any()
    else:
        assert np.isfinite(ref).all() and ref.max() < 3.4e38
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
    ok = np.isfinite(ref)
    assert np.isfinite(got[ok]).all() and (np.abs(got[ok] - ref[ok]) <= 1e-5 * ref[ok]).all()
