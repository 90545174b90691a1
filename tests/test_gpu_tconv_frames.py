"""GPU parity of the temporal convolution on tiles of frames x positions: every shape of tile, positions and channels that do not
divide by the tile's, an odd number of K-steps, fewer frames than the tile's, several groups of frames with and without a ragged
last one, batches; without and with a cache.  Bars as in test_gpu_tconv.py.  test_host_tconv_frames.py asserts that each row takes
the kernel it names."""
import pytest

from tests.test_gpu_tconv_forms import test_kernel as _check

ROWS = [                                   # kernel, B, T, HW, D
    ("3 frames", 1, 3, 1203, 1504), ("3 frames", 2, 3, 900, 1120), ("3 frames", 2, 2, 1111, 1056),
    ("5 frames", 1, 5, 700, 1504), ("5 frames", 1, 4, 1001, 1120),
    ("7 frames", 1, 7, 900, 1120), ("7 frames", 1, 6, 1000, 1056), ("7 frames", 2, 7, 401, 1184), ("7 frames", 1, 21, 301, 1184),
    ("7 frames", 1, 13, 470, 992),
]
# row tiles of the two large kernels with whole K-steps
ROW_TILES = [("256x256", 1, 5, 3300, 608), ("long", 1, 9, 1100, 736)]


@pytest.mark.gpu
@pytest.mark.parametrize("kernel,B,T,HW,D", ROWS + ROW_TILES)
def test_frames(kernel, B, T, HW, D):
    _check(kernel, B, T, HW, D)
