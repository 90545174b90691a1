"""Which kernel the temporal convolution takes (csrc/tconv_tiles.hpp), compiled with g++ and run here."""
import os
import subprocess

import pytest

from tests.test_gpu_tconv_forms import ROWS
from tests.test_gpu_tconv_frames import ROW_TILES, ROWS as FRAME_ROWS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = tmp_path_factory.mktemp("forms") / "host_tconv_forms"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", "-fsanitize=undefined", "-fno-sanitize-recover",
                    os.path.join(ROOT, "tests", "host_tconv_forms.cpp"), "-o", str(out)], check=True)
    return str(out)


def _chosen(exe, calls):
    """The kernels of calls (B, T, HW, D, cache, num_cu)."""
    args = [str(v) for call in calls for v in call]
    return subprocess.run([exe, *args], stdout=subprocess.PIPE, text=True, check=True).stdout.splitlines()


def test_choice_is_the_cheapest(exe):
    res = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0 and res.stdout.startswith("OK"), res.stdout


@pytest.mark.parametrize("rows", [ROWS, FRAME_ROWS, ROW_TILES])
def test_rows_of_the_gpu_tests_take_their_kernels(exe, rows):
    for cache in (0, 1):
        assert _chosen(exe, [(B, T, HW, D, cache, 256) for _, B, T, HW, D in rows]) == [r[0] for r in rows]


def test_rows_of_the_gpu_tests_cover_the_kernels():
    forms = {"64x64", "128x128", "256x128", "256x256", "long"}
    assert {(r[0], r[4] % 32 != 0) for r in ROWS} == {(k, t) for k in forms for t in (False, True)}
    assert {r[0] for r in FRAME_ROWS} == {"3 frames", "5 frames", "7 frames"}
    assert {r[0] for r in ROW_TILES} == {"256x256", "long"} and all(r[4] % 32 == 0 for r in ROW_TILES)


def test_measured_choices(exe):
    """Calls measured on all kernels (us: 256x256, 256x128, 128x128, 64x64, long, frame tiles): the fastest, or within 2 % of it."""
    calls = [((1, 3, 1200, 1920, 0, 256), {"3 frames"}),
             ((1, 3, 1560, 2240, 1, 256), {"3 frames"}),        # 138 189 177 293 131 101
             ((1, 21, 1560, 2240, 0, 256), {"7 frames"}),       # 809 1003 1204 2227 831 758
             ((1, 5, 752, 2240, 0, 256), {"5 frames"}),         # 120 (the fastest on row tiles) 86
             ((1, 1, 1560, 2240, 0, 256), {"128x128"}),         # 51.6 49.2 31.4 41.9 47.6
             ((1, 3, 5526, 1880, 1, 256), {"256x256"}),         # 441 509 597 1091 457
             ((1, 3, 1400, 1800, 0, 256), {"256x128"}),         # 138 114 149 246 136
             ((1, 3, 3160, 72, 0, 256), {"64x64"}),             # 17.8 14.3 9.1 6.4 15.9
             ((1, 3, 449, 96, 1, 256), {"64x64", "128x128"}),   # frame tiles 15.3, row tiles 7.1
             ((1, 9, 2250, 480, 1, 256), {"long", "256x256"}),  # row tiles 41, frame tiles 63
             ((1, 3, 1560, 2232, 1, 256), {"256x256"})]         # no whole K-steps: no frame tiles
    for got, (call, fastest) in zip(_chosen(exe, [c for c, _ in calls]), calls):
        assert got in fastest, (call, got)
