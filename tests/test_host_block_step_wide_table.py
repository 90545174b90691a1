"""The one-launch block step of d = 112 and 128 with a full rotation table requests the table rows of its first two tiles of Q with the tiles, into
members that the rotator's constructor leaves unset.  Nothing may be written over them before they are used: the kernel is compiled as it is and with those members
given a value by the constructor, and both have to load the same."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2509_24695_amd import build

ARGS = ("const uint16_t *, const uint16_t *, const uint16_t *, uint16_t *, RopeArg, TokStrides, int, int, int, int, const float *, const float *, float *, "
        "float *, float, void *, unsigned long long, uint32_t, int, WideRoles")
MEMBERS = "f32x4 cs[DEPTH][STEPS][2];"


def _loads(folder, valued):
    """{kernel: 16-byte loads through buffer resources} of the four forms with a full table."""
    csrc = shutil.copytree(build.CSRC, folder / "csrc")
    text = (csrc / "rope.hpp").read_text()
    assert text.count(MEMBERS) == 1
    if valued:
        (csrc / "rope.hpp").write_text(text.replace(MEMBERS, MEMBERS[:-1] + " = {};"))
    forms = [f"template __global__ void sv::block_step_mfma_wide<kRopeTable, {nt}, {sole}>({ARGS});" for nt in ("true", "false") for sole in ("true", "false")]
    source = folder / "forms.hip"
    source.write_text('#include "csrc/block_step_wide.hpp"\nusing namespace sv;\n' + "\n".join(forms) + "\n")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-Rpass-analysis=kernel-resource-usage")]
    out = folder / "forms.s"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--offload-device-only", "-S", str(source), "-o", str(out)],
                   check=True, stderr=subprocess.DEVNULL)
    kernels = re.findall(r"^(_ZN\S+):\s*; @.*?\n(.*?)^\.Lfunc_end", out.read_text(), re.M | re.S)
    return {name: body.count("buffer_load_dwordx4") for name, body in kernels}


def test_requested_rows_of_the_table_reach_the_rotation(tmp_path):
    got = []
    for valued in (False, True):
        folder = tmp_path / str(valued)
        folder.mkdir()
        got.append(_loads(folder, valued))
    assert len(got[0]) == 4 and got[0] == got[1]
