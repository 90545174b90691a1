"""Which temporal convolutions take tiles of frames x positions (csrc/tconv_tiles.hpp), compiled with g++ and run here."""
import os
import subprocess

import pytest

from tests.test_gpu_tconv_frames import ROW_TILES, ROWS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = tmp_path_factory.mktemp("frames") / "host_tconv_frames"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", "-fsanitize=undefined", "-fno-sanitize-recover",
                    os.path.join(ROOT, "tests", "host_tconv_frames.cpp"), "-o", str(out)], check=True)
    return str(out)


def _frames(exe, calls):
    args = [str(v) for call in calls for v in call]
    return [int(x) for x in subprocess.run([exe, *args], stdout=subprocess.PIPE, text=True, check=True).stdout.split()]


def test_rule(exe):
    res = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0 and res.stdout.startswith("OK"), res.stdout


def test_rows_of_the_gpu_tests_take_their_kernels(exe):
    for cache in (0, 1):
        assert _frames(exe, [(B, T, HW, D, cache, 256) for _, B, T, HW, D in ROWS]) == [int(r[0].split()[0]) for r in ROWS]
        assert _frames(exe, [(B, T, HW, D, cache, 256) for _, B, T, HW, D in ROW_TILES]) == [0, 0]
    assert {r[0] for r in ROWS} == {"3 frames", "5 frames", "7 frames"}


def test_measured_choices(exe):
    """us on row tiles (the fastest of five kernels) and on frame tiles."""
    calls = [((1, 3, 1560, 2240, 1, 256), 3),            # 131 / 101
             ((1, 21, 1560, 2240, 0, 256), 7),           # 809 / 758
             ((1, 5, 752, 2240, 0, 256), 5),             # 120 / 86
             ((1, 3, 449, 96, 1, 256), 0),               # 7.1 / 15.3
             ((1, 9, 2250, 480, 1, 256), 0),             # 41 / 63
             ((1, 1, 1560, 2240, 0, 256), 0), ((1, 3, 1560, 2232, 1, 256), 0)]
    for got, (call, want) in zip(_frames(exe, [c for c, _ in calls]), calls):
        assert got == want, call
