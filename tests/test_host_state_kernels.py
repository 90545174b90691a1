"""Which bf16 state kernel serves a call at d = 112 and 128 (csrc/layout_rules.hpp), compiled with g++ and run here: the rows of the GPU
tests of these kernels take the ones they name."""
import os
import subprocess

import pytest

from tests import test_gpu_coop_state as coop, test_gpu_quad_state as quad

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = tmp_path_factory.mktemp("kernels") / "host_state_kernels"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", "-fsanitize=undefined", "-fno-sanitize-recover",
                    os.path.join(ROOT, "tests", "host_state_kernels.cpp"), "-o", str(out)], check=True)
    return str(out)


def _taken(exe, calls):
    """(kernel, chunks per head) of calls (d, B, H, tokens, rope, layout)."""
    args = [str(v) for call in calls for v in call]
    lines = subprocess.run([exe, *args], stdout=subprocess.PIPE, text=True, check=True).stdout.splitlines()
    return [(k, int(c)) for k, c in (line.split() for line in lines)]


def _rows(module):
    return [((d, B, H, g[0] * g[1] * g[2] - 2 * cut, rope, layout), kernel)
            for d, B, H, g, cut, layout, kernels in module.ROWS for rope, kernel in zip(module.ROPES, kernels)]


@pytest.mark.parametrize("module", [quad, coop])
def test_rows_of_the_gpu_tests_take_their_kernels(exe, module):
    rows = _rows(module)
    assert [k for k, _ in _taken(exe, [c for c, _ in rows])] == [k for _, k in rows]


def test_rows_cover_the_chunks(exe):
    """Every form of the folds behind the exchange, in every rotation and at both head dimensions: alone, up to 2, 4, 8 and more (quadrants: 4 and more)."""
    for module, name, folds in ((quad, "quad", (1, 2, 4, 16)), (coop, "coop", (1, 2, 4, 8, 32))):
        calls = [c for c, k in _rows(module) if k == name]
        seen = {(c[4], next(f for f in folds if C <= f)) for c, (_, C) in zip(calls, _taken(exe, calls))}
        assert seen >= {(r, f) for r in module.ROPES for f in folds}
        assert {(c[0], c[5]) for c in calls} == {(d, layout) for d in (112, 128) for layout in ("bhnd", "bnhd")}
    coop_112 = [c for c, k in _rows(coop) if k == "coop" and c[0] == 112]
    assert max(C for _, C in _taken(exe, coop_112)) > 8


def test_waits_are_those_of_their_kernels(exe):
    for module, name in ((quad, "quad"), (coop, "coop")):
        d, B, H, N = module.WAIT
        (kernel, chunks), = _taken(exe, [(d, B, H, N, "none", "bhnd")])
        assert kernel == name and chunks > 1
