"""GPU parity of the d = 112 apply that takes two neighbouring heads per workgroup ([B][N][H][d], even H): bit for bit the result of
the head-major call on the same state, whose kernel is held against the oracle elsewhere.  Edges of the 32-token tiles, sub-ranges,
odd H and, with a rotation, both sides of the line in head-tokens; and state and apply against the oracle, of long calls
the last pair of heads."""
import numpy as np
import pytest

import paper_2509_24695_amd as sv
import sv_workloads as wl
from oracle import linattn_oracle as orc
from sv_workloads import metrics
from tests.gpu_util import new_state, new_workspace, say, to_dev, to_host

pytestmark = pytest.mark.gpu
EPS = 1e-6


@pytest.mark.parametrize("rope,B,H,grid,cut", [
    ("none", 1, 2, (1, 1, 1), 0), ("none", 2, 4, (1, 1, 31), 0), ("none", 1, 20, (1, 3, 11), 0), ("none", 3, 3, (1, 5, 13), 1),
    ("none", 2, 6, (3, 11, 29), 5), ("none", 8, 18, (2, 9, 31), 2), ("none", 3, 100, (1, 3, 21), 0), ("none", 1, 2, (5, 41, 43), 1),
    ("axes", 1, 32, (32, 32, 32), 0), ("table", 1, 32, (32, 32, 32), 0), ("axes", 1, 32, (32, 32, 32), 1), ("table", 1, 32, (32, 32, 32), 1),
    ("axes", 2, 18, (21, 41, 37), 7), ("table", 2, 18, (21, 41, 37), 7), ("axes", 1, 302, (7, 23, 23), 3)])
def test_pairs_of_heads(rope, B, H, grid, cut):
    import torch
    d, N = 112, grid[0] * grid[1] * grid[2]
    t0, t1 = cut, N - cut // 2
    say(f"head_pairs B={B} H={H} grid={grid} rope={rope} [{t0},{t1})")
    gen = torch.Generator("cuda").manual_seed(N + H)
    tm = [torch.empty((B, N, H, d), dtype=torch.bfloat16, device="cuda").normal_(0, 0.5, generator=gen).permute(0, 2, 1, 3) for _ in range(3)]
    hm = [x.contiguous() for x in tm]
    cs = wl.rope_tables_3d_factored(*grid, d)
    dev = [torch.from_numpy(np.ascontiguousarray(t)).cuda() for t in cs]
    arg = {"none": (), "table": (torch.from_numpy(wl.expand_rope_tables(*cs)).cuda(),), "axes": (sv.Rope3D.from_tensors(*dev),)}[rope]
    sfx = {"none": "", "table": "_rope", "axes": "_rope3d"}[rope]
    ws = new_workspace(B, H, N, d)
    state, apply = getattr(sv, "sv_linattn_state" + sfx), getattr(sv, "sv_linattn_apply" + sfx)
    S, z = new_state(B, H, d)
    S2, z2 = new_state(B, H, d)
    O = torch.full_like(tm[0], float("nan"))
    P = torch.full_like(hm[0], float("nan"))
    assert H == 1 or N == 1 or O.stride(1) < O.stride(2)
    state(tm[1], tm[2], sv.desc_of(tm[1]), *arg, t0, t1, 0, S, z, ws)
    state(hm[1], hm[2], sv.desc_of(hm[1]), *arg, t0, t1, 0, S2, z2, ws)
    apply(tm[0], sv.desc_of(tm[0]), *arg, t0, t1, S, z, EPS, O)
    apply(hm[0], sv.desc_of(hm[0]), *arg, t0, t1, S, z, EPS, P)
    torch.cuda.synchronize()
    assert sv.sv_linattn_workspace_status(ws, B, H, d) == 0
    # fp32 sums in another order: 1e-5
    assert metrics.rel_l2(to_host(S), to_host(S2)) <= 1e-5 and metrics.rel_l2(to_host(z), to_host(z2)) <= 1e-5
    assert bool(torch.equal(O[:, :, t0:t1], P[:, :, t0:t1]))
    assert bool(torch.isnan(O[:, :, :t0].float()).all()) and bool(torch.isnan(O[:, :, t1:].float()).all())
    # against the oracle: all heads of short calls, the last pair of the last batch of long ones
    b0, h0 = (0, 0) if N <= 2000 else (B - 1, H - 2)
    T = wl.expand_rope_tables(*cs) if rope != "none" else None
    Q, K, V = (to_host(x[b0:, h0:]) for x in hm)
    S_ref, z_ref = orc.state(K, V, t0=t0, t1=t1, rope=T)
    tol = 1e-5 if rope == "none" else 3e-3             # rotated bf16 keys: 2^-9 / sqrt(3) per term
    assert metrics.rel_l2(to_host(S[b0:, h0:]), S_ref) <= tol and metrics.rel_l2(to_host(z[b0:, h0:]), z_ref) <= 1e-5
    O_ref = orc.apply(Q, S_ref, z_ref, EPS, t0=t0, t1=t1, rope=T)
    metrics.check(to_host(O[b0:, h0:])[:, :, t0:t1], O_ref, "bf16", "O")
