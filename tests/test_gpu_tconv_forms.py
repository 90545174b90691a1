"""GPU parity of every kernel on row tiles that tconv_form can choose for the temporal convolution, with channels that are and are not a
multiple of the K-step, an odd number of K-steps where there is one, without and with a cache.  test_host_tconv_forms.py asserts that
each row does take the kernel it names.  Bars as in test_gpu_tconv.py."""
import numpy as np
import pytest

import paper_2509_24695_amd as sv
from oracle import tconv_oracle as orc
from sv_workloads import TconvWorkload, draw_tconv
from tests.gpu_util import say, to_dev, to_host

ROWS = [                                   # kernel, B, T, HW, D
    ("64x64", 1, 3, 300, 480), ("64x64", 2, 2, 300, 24),
    ("128x128", 1, 3, 1400, 480), ("128x128", 2, 3, 1400, 232),
    ("256x128", 2, 5, 2600, 608), ("256x128", 1, 3, 1400, 904),
    ("256x256", 1, 5, 2700, 992), ("256x256", 1, 3, 3400, 1752),
    ("long", 1, 9, 2100, 480), ("long", 2, 5, 1800, 424),
]


@pytest.mark.gpu
@pytest.mark.parametrize("kernel,B,T,HW,D", ROWS)
def test_kernel(kernel, B, T, HW, D):
    import torch
    say(f"tconv form {kernel} B={B} T={T} HW={HW} D={D}")
    w = TconvWorkload("form", B=B, T=T, HW=HW, D=D, seed=2400 + D + HW, n_blocks=2)
    xb, Wb = draw_tconv(w)
    Wd, cache_ref, cache = to_dev(Wb), None, None
    for m in range(2):
        blk = np.ascontiguousarray(xb[:, m * T:(m + 1) * T])
        y = torch.full((B, T, HW, D), float("nan"), dtype=torch.bfloat16, device="cuda")
        new_cache = torch.full((B, HW, D), float("nan"), dtype=torch.bfloat16, device="cuda")
        sv.sv_tconv_block_step(to_dev(blk), Wd, cache, y, new_cache, B, T, HW, D)
        torch.cuda.synchronize()
        y_ref, cache_ref = orc.tconv_block(blk, Wb, cache_ref)
        diff = np.abs(to_host(y) - y_ref)
        assert not (diff > np.abs(y_ref) * 2.0 ** -8 + 1e-3).any() and np.isfinite(diff).all()
        assert np.array_equal(to_host(new_cache).astype(np.float64), cache_ref)
        cache = new_cache
