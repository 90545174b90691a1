"""How the one-launch block step of d = 112 and 128 is dealt and when it is used, compiled with g++ and run here; the rows of its GPU test take the
forms they name."""
import os
import subprocess

import pytest

from tests import test_gpu_block_step_wide as wide

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _compiled(folder, name):
    out = folder / name
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", "-fsanitize=undefined", "-fno-sanitize-recover",
                    os.path.join(ROOT, "tests", name + ".cpp"), "-o", str(out)], check=True)
    return str(out)


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return _compiled(tmp_path_factory.mktemp("wide"), "host_wide_step")


def _served(exe, calls):
    """(form, workgroups of a spread head, of a local head) of calls (d, B, H, tokens, rope, layout)."""
    args = [str(v) for call in calls for v in call]
    lines = subprocess.run([exe, *args], stdout=subprocess.PIPE, text=True, check=True).stdout.splitlines()
    return [(f, int(s), int(c)) for f, s, c in (line.split() for line in lines)]


def test_heads_are_dealt_once(exe):
    res = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0 and res.stdout.startswith("OK"), res.stdout


def test_rows_of_the_gpu_test_take_their_forms(exe):
    rows = [((d, B, H, g[0] * g[1] * g[2], rope, layout), form)
            for d, B, H, g, layout, forms in wide.ROWS for rope, form in zip(wide.ROPES, forms)]
    got = _served(exe, [c for c, _ in rows])
    assert [f for f, _, _ in got] == [f for _, f in rows]
    # every form of the fold, for heads on one die and for spread ones, in every rotation
    for kind in (1, 2):
        seen = {(c[4], next(f for f in (2, 4, 8, 32) if g[kind] <= f)) for (c, _), g in zip(rows, got) if g[kind] > 1}
        assert seen >= {(r, f) for r in wide.ROPES for f in (2, 4, 8, 32)}, (kind, seen)


def test_lines(exe):
    """Calls on both sides of the lines between one launch and two."""
    calls = {(112, 1, 20, 75600, "none", "bhnd"): 1, (112, 1, 20, 75600, "axes", "bhnd"): 0, (112, 1, 20, 32760, "axes", "bhnd"): 1,
             (112, 8, 16, 1560, "none", "bhnd"): 1, (112, 4, 32, 4680, "none", "bhnd"): 0, (128, 4, 32, 4680, "none", "bhnd"): 1,
             (112, 1, 20, 9360, "table", "bhnd"): 1, (112, 1, 20, 32760, "table", "bhnd"): 0, (112, 1, 20, 4680, "none", "bnhd"): 1,
             (112, 1, 20, 14040, "none", "bnhd"): 0, (112, 1, 20, 4680, "axes", "bnhd"): 1, (112, 1, 20, 14040, "axes", "bnhd"): 0, (112, 1, 2, 600, "none", "bhnd"): 1,
             (112, 1, 2, 4680, "none", "bhnd"): 0, (112, 5, 26, 2000, "none", "bhnd"): 1, (112, 5, 26, 3120, "none", "bhnd"): 0,
             (112, 5, 26, 2000, "axes", "bhnd"): 0, (112, 10, 40, 9360, "axes", "bhnd"): 1, (112, 8, 20, 4680, "none", "bnhd"): 0,
             (112, 8, 20, 1560, "table", "bhnd"): 0, (112, 8, 32, 9360, "none", "bhnd"): 1, (112, 8, 32, 9360, "axes", "bhnd"): 0}
    got = _served(exe, list(calls))
    assert {c: int(g[0] != "two") for c, g in zip(calls, got)} == calls


def test_lines_end_where_two_launches_were_measured_ahead(exe):
    """Both sides of lines that were once left open or drawn where one launch is the slower one."""
    calls = {}
    for d, rope, BH, serves, two in ((112, "none", 260, 7800, 9360), (112, "axes", 260, 4680, 6240), (112, "none", 350, 14040, 32760), (112, "axes", 400, 9360, 14040),
                                     (128, "none", 300, 7800, 14040), (112, "none", 192, 18720, 32760), (112, "none", 240, 32760, 65520), (112, "none", 146, 3900, 4680),
                                     (112, "axes", 150, 1248, 2560), (112, "axes", 160, 2560, 3120), (128, "none", 128, 15600, 32760), (128, "none", 87, 9360, 15600),
                                     (128, "none", 84, 23400, 32760), (112, "none", 20, 75600, 131040), (112, "none", 7, 1040, 1560), (112, "axes", 7, 1040, 2028),
                                     (112, "table", 7, 2028, 4680), (128, "none", 3, 1560, 2028), (128, "none", 5, 1040, 1560), (128, "axes", 5, 1560, 2028),
                                     (128, "table", 7, 1040, 1560), (128, "none", 13, 1040, 1560), (128, "none", 10, 6240, 3120), (128, "none", 16, 3120, 500000),
                                     (128, "table", 8, 1560, 4680), (128, "table", 10, 9360, 3120), (128, "table", 16, 3780, 2070), (128, "table", 17, 3780, 3120), (128, "table", 18, 3120, 2756),
                                     (128, "table", 20, 2756, 2340), (128, "table", 20, 1560, 2070), (128, "table", 22, 2070, 20000), (128, "axes", 13, 3120, 200000)):
        calls[(d, 1, BH, serves, rope, "bhnd")], calls[(d, 1, BH, two, rope, "bhnd")] = 1, 0
    for H, n, serves in ((20, 4680, 1), (20, 9360, 0), (40, 3120, 1), (40, 4680, 0), (7, 2028, 1)):
        calls[(112, 1, H, n, "none", "bnhd")] = serves
    got = _served(exe, list(calls))
    assert {c: int(g[0] != "two") for c, g in zip(calls, got)} == calls


def test_flags_of_the_two_kinds_of_heads_share_no_line(tmp_path):
    res = subprocess.run([_compiled(tmp_path, "host_wide_flags")], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0 and res.stdout.startswith("OK"), res.stdout
