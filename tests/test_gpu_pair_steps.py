"""The d = 112 apply of two heads per workgroup with one barrier per step: rotated calls on both sides of the line in head-tokens, odd and even numbers of
32-token steps per workgroup and none at all for some, and plain calls whose token rows are multiples of 1 KB, which keep two barriers."""
import pytest

from tests.test_gpu_head_pairs import test_pairs_of_heads as check_pairs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rope,B,H,grid,cut", [
    ("axes", 1, 20, (1, 58, 58), 0), ("axes", 1, 20, (1, 56, 58), 0), ("table", 1, 20, (1, 57, 58), 0), ("axes", 2, 32, (3, 19, 19), 2), ("table", 2, 64, (1, 17, 31), 1),
    ("axes", 64, 6, (1, 13, 14), 0), ("table", 16, 130, (1, 1, 33), 0), ("axes", 40, 64, (1, 3, 9), 0),
    ("none", 1, 32, (1, 3, 11), 0), ("none", 2, 32, (3, 23, 29), 3), ("none", 1, 64, (1, 1, 31), 0), ("none", 1, 34, (1, 9, 29), 0)])
def test_steps_with_one_barrier(rope, B, H, grid, cut):
    check_pairs(rope, B, H, grid, cut)
