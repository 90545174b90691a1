"""GPU parity of the temporal convolution at the edges of its tiles: odd numbers of K-steps, K tails, tiles inside the first and
the last frame (whose zero taps are left out), one-frame blocks (test_gpu_tconv_forms.py: every kernel).  Bars as in test_gpu_tconv.py: one
rounding to bf16, 2^-8 of a value plus 1e-3 for the fp32 sums."""
import numpy as np
import pytest

import paper_2509_24695_amd as sv
from oracle import tconv_oracle as orc
from sv_workloads import TconvWorkload, draw_tconv
from tests.gpu_util import say, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,HW,D,n_blocks", [
    (1, 1, 1, 8, 2), (2, 2, 3, 24, 2), (1, 3, 64, 32, 2), (1, 3, 65, 72, 2), (2, 4, 130, 56, 2),
    (1, 1, 700, 1000, 2), (2, 3, 257, 904, 2), (1, 2, 1100, 992, 1),
    (1, 3, 2600, 992, 2), (2, 2, 3100, 1016, 1), (1, 1, 9000, 736, 2),
])
def test_tile_edges(B, T, HW, D, n_blocks):
    import torch
    say(f"tconv tiles B={B} T={T} HW={HW} D={D}")
    w = TconvWorkload("edge", B=B, T=T, HW=HW, D=D, seed=2300 + D + HW, n_blocks=n_blocks)
    xb, Wb = draw_tconv(w)
    Wd, cache_ref, cache = to_dev(Wb), None, None
    for m in range(n_blocks):
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
