"""The fp32-arithmetic state kernel whose last workgroup of a head adds the partial states up: both sides of its lines in workgroups per head (16 at d = 32,
4 at d = 64, of 256 compute units), in place and from zero, in workspaces that hold anything, and replayed by a graph without preparation."""
import numpy as np
import pytest

import paper_2509_24695_amd as sv
import sv_workloads as wl
from oracle import linattn_oracle as orc
from sv_workloads import metrics
from tests.gpu_util import new_state, new_workspace, say, to_dev, to_host

pytestmark = pytest.mark.gpu


def _inputs(seed, dtype, B, H, N, d):
    _, K, V = wl.draw_tensors(seed + N + d, (B, H, N, d), 0.5, dtype)
    rng = np.random.Generator(np.random.PCG64(97))
    S0 = rng.standard_normal((B, H, d, d), dtype=np.float32)
    z0 = np.abs(rng.standard_normal((B, H, d), dtype=np.float32))
    return K, V, S0, z0


@pytest.mark.parametrize("rope", ["none", "table", "axes"])
@pytest.mark.parametrize("dtype,d,B,H,grid", [
    ("f32", 32, 1, 15, (3, 29, 31)), ("f32", 32, 1, 16, (3, 29, 31)), ("bf16", 32, 2, 8, (3, 29, 31)), ("bf16", 32, 5, 17, (1, 29, 31)), ("f32", 32, 4, 32, (2, 29, 31)),
    ("f32", 64, 1, 51, (1, 29, 31)), ("f32", 64, 2, 32, (1, 29, 31)), ("f32", 64, 5, 17, (1, 29, 31)), ("f32", 64, 4, 32, (1, 29, 31))])
def test_last_workgroup_folds(dtype, d, B, H, grid, rope):
    import torch
    N = grid[0] * grid[1] * grid[2]
    say(f"f32_last_fold {dtype} d={d} B={B} H={H} grid={grid} {rope}")
    K, V, S0, z0 = _inputs(9980, dtype, B, H, N, d)
    cs = wl.rope_tables_3d_factored(*grid, d)
    T = wl.expand_rope_tables(*cs)
    Kd, Vd = to_dev(K), to_dev(V)
    dev = [torch.from_numpy(np.ascontiguousarray(t)).cuda() for t in cs]
    arg = {"none": (), "table": (torch.from_numpy(T).cuda(),), "axes": (sv.Rope3D.from_tensors(*dev),)}[rope]
    state = getattr(sv, "sv_linattn_state" + {"none": "", "table": "_rope", "axes": "_rope3d"}[rope])
    S_ref, z_ref = orc.state(K, V, rope=T if rope != "none" else None)
    ws, dsc = new_workspace(B, H, N, d), sv.desc_of(Kd)
    first = {}
    for contents in (0, 255, 1, None):                       # None: what the last call left
        for accumulate in (0, 1):
            if contents is not None:
                ws.view(torch.uint8).fill_(contents)
            S, z = new_state(B, H, d)
            S.copy_(torch.from_numpy(S0))
            z.copy_(torch.from_numpy(z0))
            state(Kd, Vd, dsc, *arg, 0, N, accumulate, S, z, ws)
            torch.cuda.synchronize()
            assert metrics.rel_l2(to_host(S), S_ref + accumulate * S0) <= 1e-5 and metrics.rel_l2(to_host(z), z_ref + accumulate * z0) <= 1e-5    # fp32 sums
            S1, z1 = first.setdefault(accumulate, (S, z))
            assert torch.equal(S, S1) and torch.equal(z, z1)  # whichever workgroup was last


@pytest.mark.parametrize("dtype,d,H,N", [("bf16", 32, 32, 1560), ("f32", 64, 64, 1001)])
def test_replayed_without_preparation(dtype, d, H, N):
    import torch
    say(f"f32_last_fold graph {dtype} d={d} H={H} N={N}")
    K, V, _, _ = _inputs(9990, dtype, 1, H, N, d)
    Kd, Vd = to_dev(K), to_dev(V)
    dsc = sv.desc_of(Kd)
    ws = new_workspace(1, H, N, d)
    S, z = new_state(1, H, d)

    def enqueue():
        sv.sv_linattn_state(Kd, Vd, dsc, 0, N, 0, S, z, ws, stream=torch.cuda.current_stream())
        sv.sv_linattn_state(Kd, Vd, dsc, 0, N // 2, 1, S, z, ws, stream=torch.cuda.current_stream())

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        enqueue()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    S1, z1 = S.clone(), z.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        enqueue()
    for i in range(4):
        S.fill_(7.0)
        z.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(S, S1) and torch.equal(z, z1), f"replay {i}"
        enqueue()                                             # eager work in the same workspace between the replays
        torch.cuda.synchronize()
        assert torch.equal(S, S1) and torch.equal(z, z1), f"eager call {i}"
