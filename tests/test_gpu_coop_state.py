"""GPU parity of the state kernel on shared tiles (bf16, d = 112 and 128, no full table): the edges of its 64-token tiles, one workgroup
per head to many, token sub-ranges, both layouts, an update in place, more heads than can wait for each other; and a wait that
runs out leaves S and z alone."""
import numpy as np
import pytest

import paper_2509_24695_amd as sv
import sv_workloads as wl
from oracle import linattn_oracle as orc
from sv_workloads import metrics
from tests.gpu_util import new_state, new_workspace, say, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rope", ["none", "axes"])
@pytest.mark.parametrize("d,B,H,grid,cut,layout", [
    (112, 2, 33, (1, 7, 9), 0, "bhnd"), (128, 2, 33, (1, 8, 8), 0, "bhnd"), (112, 3, 30, (1, 5, 13), 0, "bnhd"),   # 63, 64, 65 tokens
    (128, 2, 40, (3, 11, 13), 5, "bhnd"), (112, 2, 40, (3, 11, 13), 3, "bnhd"), (112, 2, 65, (1, 3, 43), 1, "bhnd"),
    (112, 2, 20, (2, 16, 31), 0, "bhnd"), (128, 4, 64, (1, 1, 257), 0, "bnhd"), (112, 5, 60, (1, 1, 97), 0, "bhnd"),  # 300 heads
    (112, 1, 1, (19, 57, 71), 7, "bhnd"), (128, 1, 3, (17, 41, 49), 0, "bhnd")])
def test_shared_tiles(d, B, H, grid, cut, layout, rope):
    import torch
    N = grid[0] * grid[1] * grid[2]
    t0, t1 = cut, N - cut
    say(f"coop_state d={d} B={B} H={H} grid={grid} [{t0},{t1}) {layout} {rope}")
    _, K, V = wl.draw_tensors(9800 + N + d, (B, H, N, d), 0.5, "bf16")
    rng = np.random.Generator(np.random.PCG64(79))
    S0 = rng.standard_normal((B, H, d, d), dtype=np.float32)
    z0 = np.abs(rng.standard_normal((B, H, d), dtype=np.float32))
    cs = wl.rope_tables_3d_factored(*grid, d)
    T = wl.expand_rope_tables(*cs)
    Kd, Vd = to_dev(K), to_dev(V)
    if layout == "bnhd":
        Kd, Vd = (x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for x in (Kd, Vd))
    dev = [torch.from_numpy(np.ascontiguousarray(t)).cuda() for t in cs]
    arg = (sv.Rope3D.from_tensors(*dev),) if rope == "axes" else ()
    state = sv.sv_linattn_state_rope3d if rope == "axes" else sv.sv_linattn_state
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


def test_wait_that_runs_out_stores_nothing():
    import torch
    B, H, N, d = 2, 40, 900, 112
    say("coop_state wait limit 0")
    _, K, V = wl.draw_tensors(9900, (B, H, N, d), 0.5, "bf16")
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
