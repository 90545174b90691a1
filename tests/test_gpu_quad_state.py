"""GPU parity of the quadrant state kernel (bf16, d = 112 and 128, short ranges): one chunk to sixteen per head, the edges of its
tiles (16 and 32 tokens, 128 and 256 per round of a workgroup), token sub-ranges, both layouts, an update in place; the next
sizes on the kernels of whole rows; and a wait that runs out leaves S and z alone.  test_host_state_kernels.py asserts that each
row takes the kernels it names."""
import numpy as np
import pytest

import paper_2509_24695_amd as sv
import sv_workloads as wl
from oracle import linattn_oracle as orc
from sv_workloads import metrics
from tests.gpu_util import new_state, new_workspace, say, to_dev, to_host

ROPES = ("none", "table", "axes")
QUAD = ("quad",) * 3
ROWS = [                                   # d, B, H, grid, tokens cut off at both ends, layout; the kernels without rotation, with a table, with axes
    (112, 1, 2, (1, 1, 1), 0, "bhnd", QUAD), (128, 1, 1, (1, 3, 5), 0, "bhnd", QUAD), (112, 1, 3, (1, 16, 16), 0, "bhnd", QUAD),
    (112, 2, 1, (1, 1, 257), 0, "bhnd", QUAD), (128, 1, 2, (3, 41, 37), 7, "bhnd", QUAD), (112, 1, 2, (3, 41, 37), 3, "bhnd", QUAD),
    (112, 1, 5, (2, 25, 31), 1, "bnhd", ("coop", "quad", "quad")), (112, 1, 8, (2, 25, 31), 1, "bnhd", QUAD), (112, 2, 8, (1, 30, 33), 0, "bnhd", QUAD),
    (128, 2, 10, (1, 29, 31), 0, "bnhd", QUAD), (112, 1, 32, (1, 25, 31), 2, "bhnd", ("coop", "quad", "quad")), (112, 1, 32, (1, 20, 31), 2, "bhnd", QUAD), (128, 2, 32, (1, 17, 31), 0, "bhnd", QUAD),
    (112, 2, 32, (1, 9, 31), 0, "bnhd", QUAD), (112, 1, 40, (1, 9, 31), 0, "bhnd", ("coop", "rows", "coop")),
    (128, 1, 65, (1, 9, 31), 0, "bhnd", ("coop", "rows", "coop"))]


def check_state(name, d, B, H, grid, cut, layout, rope, seeds):
    """State of tokens [cut, N - cut) in place of, and added to, a carried one, against the oracle."""
    import torch
    N = grid[0] * grid[1] * grid[2]
    t0, t1 = cut, N - cut
    say(f"{name} d={d} B={B} H={H} grid={grid} [{t0},{t1}) {layout} {rope}")
    _, K, V = wl.draw_tensors(seeds[0] + N + d, (B, H, N, d), 0.5, "bf16")
    rng = np.random.Generator(np.random.PCG64(seeds[1]))
    S0 = rng.standard_normal((B, H, d, d), dtype=np.float32)
    z0 = np.abs(rng.standard_normal((B, H, d), dtype=np.float32))
    cs = wl.rope_tables_3d_factored(*grid, d)
    T = wl.expand_rope_tables(*cs)
    Kd, Vd = to_dev(K), to_dev(V)
    if layout == "bnhd":
        Kd, Vd = (x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for x in (Kd, Vd))
    dev = [torch.from_numpy(np.ascontiguousarray(t)).cuda() for t in cs]
    arg = {"none": (), "table": (torch.from_numpy(T).cuda(),), "axes": (sv.Rope3D.from_tensors(*dev),)}[rope]
    state = getattr(sv, "sv_linattn_state" + {"none": "", "table": "_rope", "axes": "_rope3d"}[rope])
    S, z = new_state(B, H, d)
    S.copy_(torch.from_numpy(S0))
    z.copy_(torch.from_numpy(z0))
    ws, dsc = new_workspace(B, H, N, d), sv.desc_of(Kd)
    S_ref, z_ref = orc.state(K, V, t0=t0, t1=t1, rope=T if rope != "none" else None)
    tol = 1e-5 if rope == "none" else 3e-3             # rotated bf16 keys: 2^-9 / sqrt(3) per term
    state(Kd, Vd, dsc, *arg, t0, t1, 1, S, z, ws)
    torch.cuda.synchronize()
    assert metrics.rel_l2(to_host(S), S0 + S_ref) <= tol and metrics.rel_l2(to_host(z), z0 + z_ref) <= 1e-5
    state(Kd, Vd, dsc, *arg, t0, t1, 0, S, z, ws)
    torch.cuda.synchronize()
    assert sv.sv_linattn_workspace_status(ws, B, H, d) == 0
    assert metrics.rel_l2(to_host(S), S_ref) <= tol and metrics.rel_l2(to_host(z), z_ref) <= 1e-5


def check_wait_that_runs_out(name, d, B, H, N, seed):
    import torch
    say(f"{name} wait limit 0")
    _, K, V = wl.draw_tensors(seed, (B, H, N, d), 0.5, "bf16")
    Kd, Vd = to_dev(K), to_dev(V)
    S, z = new_state(B, H, d)
    S.fill_(3.0)
    z.fill_(4.0)
    ws = new_workspace(B, H, N, d)
    try:
        sv.sv_linattn_set_wait_limit(0)
        sv.sv_linattn_state(Kd, Vd, sv.desc_of(Kd), 0, N, 0, S, z, ws)
        torch.cuda.synchronize()
    finally:
        sv.sv_linattn_set_wait_limit(-1)
    assert sv.sv_linattn_workspace_status(ws, B, H, d) == 1
    assert bool((S == 3.0).all()) and bool((z == 4.0).all())


WAIT = (112, 1, 20, 900)                   # d, B, H, tokens: quad


@pytest.mark.gpu
@pytest.mark.parametrize("rope", ROPES)
@pytest.mark.parametrize("d,B,H,grid,cut,layout,kernels", ROWS)
def test_quadrants(d, B, H, grid, cut, layout, kernels, rope):
    check_state("quad_state", d, B, H, grid, cut, layout, rope, (9600, 78))


@pytest.mark.gpu
def test_wait_that_runs_out_stores_nothing():
    check_wait_that_runs_out("quad_state", *WAIT, 9700)
