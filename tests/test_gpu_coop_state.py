"""GPU parity of the state kernel on shared tiles (bf16, d = 112 and 128, no full table): the edges of its 64-token tiles, one workgroup
per head to many, token sub-ranges, both layouts, an update in place, more heads than can wait for each other; and a wait that
runs out leaves S and z alone.  test_host_state_kernels.py asserts that each row takes the kernel it names."""
import pytest

from tests.test_gpu_quad_state import check_state, check_wait_that_runs_out

ROPES = ("none", "axes")
COOP = ("coop",) * 2
ROWS = [                                   # d, B, H, grid, tokens cut off at both ends, layout; the kernels without rotation, with axes
    (112, 2, 33, (1, 7, 9), 0, "bhnd", COOP), (128, 2, 33, (1, 8, 8), 0, "bhnd", COOP), (112, 3, 30, (1, 5, 13), 0, "bnhd", COOP),   # 63, 64, 65 tokens
    (128, 2, 40, (3, 11, 13), 5, "bhnd", COOP), (112, 2, 40, (3, 11, 13), 3, "bnhd", COOP), (112, 2, 65, (1, 3, 43), 1, "bhnd", COOP),
    (112, 2, 20, (2, 16, 31), 0, "bhnd", COOP), (128, 4, 64, (1, 1, 257), 0, "bnhd", COOP), (112, 5, 60, (1, 1, 97), 0, "bhnd", COOP),  # 300 heads
    (112, 1, 3, (19, 37, 41), 7, "bhnd", COOP), (128, 1, 3, (17, 41, 49), 0, "bhnd", COOP),              # 32 chunks per head
    (112, 1, 1, (19, 57, 71), 7, "bhnd", ("rows", "rows"))]                                              # past 2 048 tokens per workgroup
WAIT = (112, 2, 40, 900)                   # d, B, H, tokens: coop


@pytest.mark.gpu
@pytest.mark.parametrize("rope", ROPES)
@pytest.mark.parametrize("d,B,H,grid,cut,layout,kernels", ROWS)
def test_shared_tiles(d, B, H, grid, cut, layout, kernels, rope):
    check_state("coop_state", d, B, H, grid, cut, layout, rope, (9800, 79))


@pytest.mark.gpu
def test_wait_that_runs_out_stores_nothing():
    check_wait_that_runs_out("coop_state", *WAIT, 9900)
