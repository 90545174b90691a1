"""The convolution's products are inline assembly (tc_mfma, csrc/tconv_mfma.hpp), which the compiler schedules around without knowing what the
matrix instructions need.  Here its output is read for that (numbers of wait states: what the compiler leaves after and before the same products as
builtins): two between a vector write of an operand and its use, eight between a product and anything but a product that reads what it wrote; an
accumulator is used again no sooner than four products later and none is moved in a loop."""
import os
import re
import subprocess

import pytest

from paper_2509_24695_amd import build

MFMA = "v_mfma_f32_16x16x32_bf16"
_REG = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")


def _regs(text):
    out = set()
    for kind, one, lo, hi in _REG.findall(text):
        out |= {(kind, int(one))} if one else {(kind, i) for i in range(int(lo), int(hi) + 1)}
    return out


def _kernels(asm):
    """{name: instructions} of the kernels that have such products."""
    out = {}
    for name, body in re.findall(r"^(_ZN\S+):\s*; @.*?\n(.*?)^\.Lfunc_end", asm, re.M | re.S):
        if MFMA not in body:
            continue
        lines = (x.split(";")[0].strip() for x in body.split("\n"))
        out[name] = [x for x in lines if x and not x.startswith(".") and not x.endswith(":")]
    return out


def _hazards(ins):
    """Complaints about a run of instructions."""
    state = products = 0
    written, produced, bad = {}, {}, []          # register -> wait state of the last vector write; -> (state, product) that wrote it
    for x in ins:
        op, _, rest = x.partition(" ")
        operands = [o.strip() for o in rest.split(", ")]
        if op == "s_nop":
            state += int(operands[0], 0) + 1
            continue
        state += 1
        if op == MFMA:
            products += 1
            acc, sources = _regs(operands[0]), _regs(operands[1]) | _regs(operands[2])
            assert acc == _regs(operands[3]) and all(k == "a" for k, _ in acc) and all(k == "v" for k, _ in sources), x
            bad += [f"{x}: {r} written {state - written[r]} states before" for r in acc | sources if state - written.get(r, -9) <= 2]
            bad += [f"{x}: {r} of {products - produced[r][1]} products before" for r in acc if r in produced and products - produced[r][1] < 4]
            produced.update({r: (state, products) for r in acc})
            continue
        used = _regs(rest)
        bad += [f"{x}: {r} of a product {state - produced[r][0]} states before" for r in used if r in produced and state - produced[r][0] <= 8]
        if op.startswith("v_") and not op.startswith("v_cmp"):
            for r in _regs(operands[0]):
                written[r] = state
                produced.pop(r, None)
    return bad


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "sv_tconv.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-Rpass-analysis=kernel-resource-usage")]
    source = next(s for s in build.SOURCES if s.endswith("sv_tconv.hip"))
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--offload-device-only", "-S", source, "-o", str(out)],
                   check=True, stderr=subprocess.DEVNULL)
    return _kernels(out.read_text())


def test_products_are_scheduled_as_they_need(kernels):
    assert sum("tconv_frames" in k for k in kernels) == 5 and sum("tconv_mfma" in k for k in kernels) == 7
    for name, ins in kernels.items():
        at = [i for i, x in enumerate(ins) if x.startswith(MFMA)]
        loop = ins[at[0]:at[-1] + 1]
        assert not [x for x in loop if x.startswith("v_accvgpr")], name
        assert _hazards(loop + loop) == [] and _hazards(ins) == [], name


def test_the_reader_sees_planted_hazards(kernels):
    ins = next(v for k, v in kernels.items() if "tconv_frames" in k)
    at = [i for i, x in enumerate(ins) if x.startswith(MFMA)]
    first, last = at[5], at[-1]
    acc, a = (o.strip() for o in ins[first].partition(" ")[2].split(", ")[:2])
    one = "v%d" % min(r for _, r in _regs(a))
    plant = lambda i, x: _hazards(ins[:i] + [x] + ins[i:])
    assert plant(first, f"v_mov_b32_e32 {one}, 0") and plant(first - 1, f"v_add_u32_e32 {one}, 1, {one}")
    assert not _hazards(ins[:first] + [f"v_mov_b32_e32 {one}, 0", "s_nop 1"] + ins[first:])
    done = "a%d" % min(r for _, r in _regs(ins[last].partition(" ")[2].split(", ")[0]))
    assert plant(last + 1, f"v_accvgpr_read_b32 v0, {done}")
    assert plant(first + 1, ins[first])
