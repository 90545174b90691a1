"""One workgroup, or four with a quarter of the state each, per head in the fp32-arithmetic state kernel: sixteen waves at d = 32 (tiles of 32 tokens, of 16 with
a rotation, 512 or 256 to a round), eight at d >= 64 (tiles of 8, 64 to a round; at d = 112 and 128 two groups that share the state, 16 to a round).  The
edges of their rounds, and both sides of the lines where several workgroups take over, against the oracle."""
import pytest

from tests.test_gpu_f32_mfma import _layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rope", ["none", "table", "axes"])
@pytest.mark.parametrize("dtype,d,heads,grid,cut", [
    ("f32", 32, 3, (1, 1, 31), 0), ("f32", 32, 2, (1, 1, 257), 0), ("f32", 32, 2, (1, 16, 32), 0), ("f32", 32, 2, (1, 19, 27), 0),
    ("f32", 32, 2, (1, 32, 36), 0), ("f32", 32, 17, (1, 28, 32), 0), ("f32", 32, 2, (1, 31, 33), 1), ("bf16", 32, 2, (1, 30, 42), 3),
    ("bf16", 32, 33, (1, 28, 32), 0), ("f32", 64, 2, (1, 16, 16), 0), ("f32", 64, 2, (1, 1, 257), 0),
    ("f32", 112, 2, (1, 6, 8), 0), ("f32", 128, 9, (1, 7, 7), 0), ("f32", 112, 2, (1, 8, 8), 0), ("f32", 112, 2, (1, 5, 13), 0), ("f32", 128, 9, (1, 6, 16), 0), ("f32", 112, 33, (1, 8, 16), 1),
    ("f32", 32, 5, (1, 20, 32), 0), ("f32", 32, 5, (1, 26, 32), 0), ("f32", 32, 3, (1, 17, 49), 0), ("f32", 32, 40, (1, 16, 32), 0), ("f32", 32, 20, (1, 3, 171), 0),
    ("bf16", 32, 9, (1, 28, 32), 0), ("bf16", 32, 40, (1, 20, 32), 0), ("bf16", 32, 20, (1, 3, 235), 0), ("f32", 64, 3, (1, 12, 16), 0), ("f32", 64, 3, (1, 1, 193), 0)])
def test_one_workgroup_per_head(dtype, d, heads, grid, cut, rope):
    _layer(dtype, d, 1, heads, grid, rope, cut, grid[0] * grid[1] * grid[2] - cut)
