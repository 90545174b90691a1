"""GPU: factored rotation tables at d = 64 with the pairs split among the axes in fours (two 16-byte lookups per chunk) and otherwise (four of
8 bytes): state, apply and block step bit for bit those of the full table they expand to."""
import numpy as np
import pytest

import paper_2509_24695_amd as sv
import sv_workloads as wl
from tests.gpu_util import new_state, new_workspace, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("split", [(8, 12, 12), (4, 4, 24), (24, 4, 4), (9, 12, 11), (8, 13, 11), (6, 14, 12), (1, 1, 30)])
@pytest.mark.parametrize("B,H,grid", [(1, 2, (3, 7, 11)), (2, 4, (5, 16, 33)), (1, 8, (3, 37, 29))])
def test_splits(split, B, H, grid):
    import torch
    d, N = 64, grid[0] * grid[1] * grid[2]
    say(f"rope3d_splits {split} B={B} H={H} grid={grid}")
    Q, K, V = (to_dev(x) for x in wl.draw_tensors(9950 + N, (B, H, N, d), 0.5, "bf16"))
    rng = np.random.Generator(np.random.PCG64(80))
    cs = []
    for n, p in zip(grid, split):
        a = rng.uniform(-np.pi, np.pi, (n, p))
        cs.append(np.stack([np.cos(a), np.sin(a)], -1).astype(np.float32))
    f, r, c = np.unravel_index(np.arange(N), grid)
    T = torch.from_numpy(np.concatenate([cs[0][f], cs[1][r], cs[2][c]], 1)).cuda()
    dev = [torch.from_numpy(t).cuda() for t in cs]
    r3 = sv.Rope3D.from_tensors(*dev)
    dsc, ws = sv.desc_of(Q), new_workspace(B, H, N, d)
    got = []
    for sfx, arg in (("_rope", T), ("_rope3d", r3)):
        for cut in (0, 5):
            S, z = new_state(B, H, d)
            O = torch.full_like(Q, float("nan"))
            getattr(sv, "sv_linattn_state" + sfx)(K, V, dsc, arg, cut, N - cut, 0, S, z, ws)
            getattr(sv, "sv_linattn_apply" + sfx)(Q, dsc, arg, cut, N - cut, S, z, 1e-6, O)
            got += [S, z, O[:, :, cut:N - cut].contiguous()]
        S, z = new_state(B, H, d)
        S.zero_()
        z.zero_()
        O = torch.full_like(Q, float("nan"))
        getattr(sv, "sv_block_linattn_step" + sfx)(Q, K, V, dsc, arg, S, z, 1e-6, O, ws)
        torch.cuda.synchronize()
        got += [S, z, O]
    n = len(got) // 2
    assert not any(bool(torch.isnan(x.float()).any()) for x in got)
    assert all(torch.equal(a, b) for a, b in zip(got[:n], got[n:]))
