"""GPU parity of the kernels with fp32 arithmetic on the matrix cores (fp32 tokens at every d, bf16 at d = 32) at the
edges of their tiles (16 and 32 tokens, 64 and 128 per workgroup), on token sub-ranges, with more heads than workgroups
fit at once, and where the factored tables are too large for them and the plain kernels run instead."""
import numpy as np
import pytest

import paper_2509_24695_amd as sv
import sv_workloads as wl
from oracle import linattn_oracle as orc
from sv_workloads import metrics
from tests.gpu_util import new_state, new_workspace, say, to_dev, to_host

pytestmark = pytest.mark.gpu


def _layer(dtype, d, B, H, grid, rope, t0, t1):
    import torch
    N = grid[0] * grid[1] * grid[2]
    say(f"f32_mfma {dtype} d={d} B={B} H={H} grid={grid} rope={rope} [{t0},{t1})")
    Q, K, V = wl.draw_tensors(9900 + N + d, (B, H, N, d), 0.5, dtype)
    cs = wl.rope_tables_3d_factored(*grid, d)
    T = wl.expand_rope_tables(*cs)
    Qd, Kd, Vd = to_dev(Q), to_dev(K), to_dev(V)
    dsc, ws = sv.desc_of(Qd), new_workspace(B, H, N, d)
    S, z = new_state(B, H, d)
    O = torch.full_like(Qd, float("nan"))
    dev = [torch.from_numpy(np.ascontiguousarray(t)).cuda() for t in cs]
    arg = {"none": (), "table": (torch.from_numpy(T).cuda(),), "axes": (sv.Rope3D.from_tensors(*dev),)}[rope]
    sfx = {"none": "", "table": "_rope", "axes": "_rope3d"}[rope]
    getattr(sv, "sv_linattn_state" + sfx)(Kd, Vd, dsc, *arg, t0, t1, 0, S, z, ws)
    getattr(sv, "sv_linattn_apply" + sfx)(Qd, dsc, *arg, t0, t1, S, z, 1e-6, O)
    torch.cuda.synchronize()
    S_ref, z_ref = orc.state(K, V, t0=t0, t1=t1, rope=T if rope != "none" else None)
    O_ref = orc.apply(Q, S_ref, z_ref, 1e-6, t0=t0, t1=t1, rope=T if rope != "none" else None)
    # everything but the output's storage is fp32: 1e-5 as for any fp32 sum here, also for rotated keys
    assert metrics.rel_l2(to_host(S), S_ref) <= 1e-5 and metrics.rel_l2(to_host(z), z_ref) <= 1e-5
    metrics.check(to_host(O)[:, :, t0:t1], O_ref, dtype, "O")
    outside = torch.cat([O[:, :, :t0], O[:, :, t1:]], dim=2)
    assert bool(torch.isnan(outside.float()).all())


@pytest.mark.parametrize("dtype,d", [("f32", 32), ("f32", 64), ("f32", 112), ("f32", 128), ("bf16", 32)])
@pytest.mark.parametrize("rope", ["none", "table", "axes"])
@pytest.mark.parametrize("B,H,grid,cut", [(1, 1, (1, 1, 1), 0), (2, 3, (1, 5, 3), 0), (1, 2, (1, 4, 4), 0), (1, 3, (1, 1, 17), 1),
                                          (1, 2, (2, 8, 8), 1), (2, 2, (3, 19, 23), 5)])
def test_tile_edges(B, H, grid, cut, rope, dtype, d):
    N = grid[0] * grid[1] * grid[2]
    _layer(dtype, d, B, H, grid, rope, cut, N - cut)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 32)])
def test_more_heads_than_fit_at_once(dtype, d):
    _layer(dtype, d, 10, 160, (1, 5, 9), "axes", 0, 45)


@pytest.mark.parametrize("dtype,d", [("f32", 112), ("bf16", 32)])
def test_tables_past_the_lds_take_the_plain_kernels(dtype, d):
    _layer(dtype, d, 1, 2, (1, 1, 900), "axes", 3, 900)
