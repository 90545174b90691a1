"""Which kernel the temporal convolution takes (csrc/tconv_tiles.hpp), compiled with g++ and run here."""
import os
import subprocess

import pytest

from tests.test_gpu_tconv_forms import ROWS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = tmp_path_factory.mktemp("forms") / "host_tconv_forms"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", "-fsanitize=undefined", "-fno-sanitize-recover",
                    os.path.join(ROOT, "tests", "host_tconv_forms.cpp"), "-o", str(out)], check=True)
    return str(out)


def _chosen(exe, calls):
    args = [str(v) for call in calls for v in call]
    return subprocess.run([exe, *args], stdout=subprocess.PIPE, text=True, check=True).stdout.split()


def test_choice_is_the_cheapest(exe):
    res = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0 and res.stdout.startswith("OK"), res.stdout


def test_rows_of_the_gpu_test_take_their_kernels(exe):
    for cache in (0, 1):
        assert _chosen(exe, [(B * T * HW, D, T, cache, 256) for _, B, T, HW, D in ROWS]) == [r[0] for r in ROWS]
    assert {r[0] for r in ROWS} == {"64x64", "128x128", "256x128", "256x256", "long"}
    assert {(r[0], r[4] % 32 != 0) for r in ROWS} == {(k, t) for k in {r[0] for r in ROWS} for t in (False, True)}


def test_measured_choices(exe):
    """Calls measured on all kernels (us: 256x256, 256x128, 128x128, 64x64, long): the fastest, or within 2 % of it."""
    calls = [((3600, 1920, 3, 0, 256), {"long"}),            # 110.4 111.4 109.9 171.9 103.1
             ((4680, 2240, 3, 1, 256), {"256x256"}),         # six calls: 829-834 us on six devices; long 812-846
             ((1560, 2240, 1, 0, 256), {"128x128"}),         # 51.6 49.2 31.4 41.9 47.6
             ((32760, 2240, 21, 0, 256), {"256x256"}),       # 789 1271 1204 2051 839
             ((16578, 1880, 3, 1, 256), {"256x256"}),        # 441 509 597 1091 457
             ((4200, 1800, 3, 0, 256), {"256x128"}),         # 138 114 149 246 136
             ((9480, 72, 3, 0, 256), {"64x64"}),             # 17.8 14.3 9.1 6.4 15.9
             ((9360, 640, 3, 0, 256), {"128x128"})]          # 46.7 43.9 38.7 51.5 43.8
    for got, (call, fastest) in zip(_chosen(exe, [c for c, _ in calls]), calls):
        assert got in fastest, (call, got)
