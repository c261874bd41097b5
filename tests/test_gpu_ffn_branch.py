"""GPU parity of ConvFFN's depth-wise branch as a launch of its own at the edges of its strips, and of the one-launch
kernels on small images (bands of one to three rows), through the whole network against the CPU oracle; the bars are tests/test_gpu_ffn.py's."""
import pytest

from paper_2503_06671_amd import workloads as wk
from tests.test_gpu_ffn import check_ffn

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
