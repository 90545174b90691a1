"""GPU parity of the temporal convolution on tiles of frames x positions: every shape of tile, positions and channels that do not
divide by the tile's, an odd number of K-steps, fewer frames than the tile's, several groups of frames with and without a ragged
last one, batches; without and with a cache.  Bars as in test_gpu_tconv.py.  test_host_tconv_forms.py asserts that each row takes
the kernel it names."""
import pytest

import paper_2509_24695_amd as sv
from tests.gpu_util import say
from tests.test_gpu_tconv_forms import test_kernel as _check

ROWS = [                                   # kernel, B, T, HW, D
    ("3 frames", 1, 3, 1203, 1504), ("3 frames", 2, 3, 900, 1120), ("3 frames", 2, 2, 1111, 1056),
    ("5 frames", 1, 5, 700, 1504), ("5 frames", 1, 4, 1001, 1120),
    ("7 frames", 1, 7, 900, 1120), ("7 frames", 1, 6, 1000, 1056), ("7 frames", 2, 7, 401, 1184), ("7 frames", 1, 21, 301, 1184),
    ("7 frames", 1, 13, 470, 992),
]
# row tiles of the two large kernels with whole K-steps
ROW_TILES = [("256x256", 1, 5, 3300, 608), ("long", 1, 9, 1100, 992)]


@pytest.mark.gpu
@pytest.mark.parametrize("kernel,B,T,HW,D", ROWS + ROW_TILES)
def test_frames(kernel, B, T, HW, D):
    _check(kernel, B, T, HW, D)


@pytest.mark.gpu
@pytest.mark.parametrize("kernel,B,T,HW,D", [r for r in ROWS if r[4] // 32 % 2])
def test_step_past_the_last_adds_nothing(kernel, B, T, HW, D):
    """An odd number of K-steps: the loop's extra one multiplies zeros with zeros, so a weight of the last 32 channels that overflowed shows as
    the infinity that its products are, in its own output channel alone."""
    import torch
    say(f"tconv frames past the last step {kernel} B={B} T={T} HW={HW} D={D}")
    gen = torch.Generator("cuda").manual_seed(D)
    x = torch.randn((B, T, HW, D), generator=gen, device="cuda").to(torch.bfloat16)
    x[..., D - 1].masked_fill_(x[..., D - 1] == 0, 1.0)
    W = (torch.randn((3, D, D), generator=gen, device="cuda") / (3 * D) ** 0.5).to(torch.bfloat16)
    y, want = torch.empty_like(x), torch.empty_like(x)
    sv.sv_tconv_block_step(x, W, None, want, None, B, T, HW, D)
    W[1, 5, D - 1] = float("inf")
    sv.sv_tconv_block_step(x, W, None, y, None, B, T, HW, D)
    torch.cuda.synchronize()
    want[..., 5] = x[..., D - 1] * float("inf")
    assert torch.equal(y, want)
