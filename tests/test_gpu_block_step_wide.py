"""GPU parity of the one-launch block step (bf16, d = 112 and 128): heads on one die, spread over the dies, both at once, a workgroup to itself, more
heads than compute units; the edges of its 64-token tiles; rotations and layouts; committing and looking ahead; a wait that runs out and a head
that is not where it should be store nothing.  test_host_wide_step.py asserts that each row takes the form it names."""
import numpy as np
import pytest

import paper_2509_24695_amd as sv
import sv_workloads as wl
from oracle import linattn_oracle as orc
from sv_workloads import metrics
from tests.gpu_util import new_state, new_workspace, say, to_dev, to_host

ROPES = ("none", "table", "axes")
ROWS = [                                   # d, B, H, grid, layout; the forms without rotation, with a table, with axes
    (112, 1, 2, (1, 1, 1), "bhnd", ("sole",) * 3), (128, 1, 3, (1, 7, 9), "bhnd", ("sole",) * 3), (112, 1, 9, (1, 8, 8), "bnhd", ("sole",) * 3),
    (112, 1, 9, (1, 5, 13), "bhnd", ("mixed",) * 3), (128, 1, 8, (1, 9, 15), "bhnd", ("local",) * 3), (112, 2, 4, (3, 25, 27), "bhnd", ("local",) * 3),
    (112, 1, 20, (1, 23, 37), "bhnd", ("mixed",) * 3), (128, 1, 20, (1, 23, 37), "bnhd", ("mixed",) * 3), (112, 1, 3, (2, 17, 31), "bhnd", ("spread",) * 3),
    (112, 1, 20, (1, 23, 37), "bnhd", ("spread",) * 3), (112, 1, 16, (3, 23, 31), "bhnd", ("local", "spread", "local")),
    (112, 2, 16, (1, 23, 31), "bhnd", ("local",) * 3), (112, 3, 20, (1, 15, 29), "bhnd", ("mixed",) * 3), (128, 4, 20, (1, 13, 31), "bhnd", ("local",) * 3), (112, 4, 31, (1, 11, 19), "bhnd", ("mixed",) * 3),
    (112, 1, 9, (4, 15, 31), "bhnd", ("mixed",) * 3),
    (112, 5, 26, (1, 11, 19), "bhnd", ("sole",) * 3), (128, 8, 20, (1, 11, 13), "bnhd", ("sole",) * 3), (112, 10, 30, (1, 7, 19), "bhnd", ("sole",) * 3)]


def _case(seed, d, B, H, grid, layout, rope):
    import torch
    N = grid[0] * grid[1] * grid[2]
    Q, K, V = wl.draw_tensors(seed + N + d, (B, H, N, d), 0.5, "bf16")
    rng = np.random.Generator(np.random.PCG64(seed))
    S0 = rng.standard_normal((B, H, d, d), dtype=np.float32)
    z0 = np.abs(rng.standard_normal((B, H, d), dtype=np.float32)) * 10
    cs = wl.rope_tables_3d_factored(*grid, d)
    T = wl.expand_rope_tables(*cs)
    dev = [to_dev(x) for x in (Q, K, V)]
    if layout == "bnhd":
        dev = [x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for x in dev]
    axes = [torch.from_numpy(np.ascontiguousarray(t)).cuda() for t in cs]
    arg = {"none": (), "table": (torch.from_numpy(T).cuda(),), "axes": (sv.Rope3D.from_tensors(*axes),)}[rope]
    return (Q, K, V), dev, S0, z0, T if rope != "none" else None, arg, axes


@pytest.mark.gpu
@pytest.mark.parametrize("rope", ROPES)
@pytest.mark.parametrize("d,B,H,grid,layout,forms", ROWS)
def test_block_step_wide(d, B, H, grid, layout, forms, rope):
    import torch
    say(f"block_step_wide d={d} B={B} H={H} grid={grid} {layout} {rope}")
    host, (q, k, v), S0, z0, T, arg, _keep = _case(9100, d, B, H, grid, layout, rope)
    O_ref, S_ref, z_ref = orc.block_step(*host, S0.astype(np.float64), z0.astype(np.float64), 1e-6, rope=T)
    ws, dsc = new_workspace(B, H, grid[0] * grid[1] * grid[2], d), sv.desc_of(q)
    sfx = {"none": "", "table": "_rope", "axes": "_rope3d"}[rope]
    s_tol = 1e-5 if rope == "none" else 3e-3             # rotated bf16 keys: 2^-9 / sqrt(3) per term
    outs = []
    for step in ("sv_block_linattn_lookahead", "sv_block_linattn_step"):
        S, z = new_state(B, H, d)
        S.copy_(torch.from_numpy(S0))
        z.copy_(torch.from_numpy(z0))
        O = torch.full_like(q, float("nan"))             # a row that is not written must not pass
        getattr(sv, step + sfx)(q, k, v, dsc, *arg, S, z, 1e-6, O, ws)
        torch.cuda.synchronize()
        assert sv.sv_linattn_workspace_status(ws, B, H, d) == 0
        metrics.check(to_host(O), O_ref, "bf16", step)
        if step.endswith("lookahead"):
            assert np.array_equal(to_host(S), S0) and np.array_equal(to_host(z), z0)
        else:
            assert metrics.rel_l2(to_host(S), S_ref) <= s_tol and metrics.rel_l2(to_host(z), z_ref) <= 1e-5
        outs.append(O)
    assert torch.equal(outs[0], outs[1])


@pytest.mark.gpu
@pytest.mark.parametrize("rope", ["none", "axes"])
@pytest.mark.parametrize("d,B,H,layout", [(112, 1, 32, "bhnd"), (128, 2, 32, "bhnd"), (128, 4, 32, "bnhd"), (112, 2, 64, "bhnd")])
def test_walks_are_those_of_the_state_kernel(d, B, H, layout, rope):
    """Heads on one die, as many workgroups each as the state kernel gives them: the same shares, met in the same order, make the same sums."""
    import torch
    grid = (1, 45, 68)
    N = grid[0] * grid[1] * grid[2]
    say(f"block_step_wide walks d={d} B={B} H={H} {layout} {rope}")
    _, (q, k, v), _, _, _, arg, _keep = _case(9170, d, B, H, grid, layout, rope)
    dsc, sfx, got = sv.desc_of(q), {"none": "", "axes": "_rope3d"}[rope], []
    for call in ("state", "step"):
        S, z = new_state(B, H, d)
        ws = new_workspace(B, H, N, d)
        if call == "state":
            getattr(sv, "sv_linattn_state" + sfx)(k, v, dsc, *arg, 0, N, 0, S, z, ws)
        else:
            getattr(sv, "sv_block_linattn_step" + sfx)(q, k, v, dsc, *arg, S, z, 1e-6, torch.empty_like(q), ws)
        torch.cuda.synchronize()
        got.append((S, z))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.gpu
@pytest.mark.parametrize("why", ["wait", "dies"])
@pytest.mark.parametrize("H", [16, 20])
def test_a_step_that_gives_up_stores_nothing(H, why):
    """16 heads: each on one die; 20: four of them spread, which the wrong number of dies does not concern."""
    import torch
    d, grid = 112, (1, 30, 52)
    say(f"block_step_wide gives up H={H} {why}")
    host, (q, k, v), _, _, _, _, _ = _case(9150, d, 1, H, grid, "bhnd", "none")
    S, z = new_state(1, H, d)
    S.fill_(3.0)
    z.fill_(5.0)
    O = torch.full_like(q, float("nan"))
    ws, dsc = new_workspace(1, H, grid[1] * grid[2], d), sv.desc_of(q)
    sv.sv_linattn_workspace_init(ws, 1, H, d)
    try:
        if why == "wait":
            sv.sv_linattn_set_wait_limit(0)
        else:
            sv.sv_measure_assume_dies(4)
        sv.sv_block_linattn_step(q, k, v, dsc, S, z, 1e-6, O, ws)
        torch.cuda.synchronize()
    finally:
        sv.sv_linattn_set_wait_limit(-1)
        sv.sv_measure_assume_dies(8)
    assert sv.sv_linattn_workspace_status(ws, 1, H, d) == 1
    assert bool((S == 3.0).all()) and bool((z == 5.0).all()) and bool(torch.isnan(O.float()).all())
    # and works again; the workspace's memory, which the next test may get, is left without the mark
    sv.sv_linattn_workspace_init(ws, 1, H, d)
    S.zero_()
    z.zero_()
    sv.sv_block_linattn_step(q, k, v, dsc, S, z, 1e-6, O, ws)
    torch.cuda.synchronize()
    assert sv.sv_linattn_workspace_status(ws, 1, H, d) == 0
    metrics.check(to_host(O), orc.bidirectional(*host, 1e-6)[0], "bf16", "after the refused step")
