"""GPU parity for token tensors laid out [B][N][H][d] (a projection's output as it lies in memory), where the layer
kernels deal their workgroups in another order and, at d = 112, go through the caches differently."""
import numpy as np
import pytest

import paper_2509_24695_amd as sv
import sv_workloads as wl
from oracle import linattn_oracle as orc
from sv_workloads import metrics
from tests.gpu_util import new_state, new_workspace, say, to_dev, to_host

pytestmark = pytest.mark.gpu


def _token_major(x):
    """Device tensor of the same values as x [B][H][N][d], stored [B][N][H][d]."""
    return to_dev(np.ascontiguousarray(x.transpose(0, 2, 1, 3))).permute(0, 2, 1, 3)


@pytest.mark.parametrize("d", [64, 112, 128])
@pytest.mark.parametrize("rope", ["none", "table", "axes"])
@pytest.mark.parametrize("B,H,grid", [(1, 2, (1, 1, 1)), (2, 3, (1, 7, 13)), (2, 20, (2, 19, 33))])
def test_token_major_layer_and_block(B, H, grid, rope, d):
    import torch
    N = grid[0] * grid[1] * grid[2]
    say(f"token_major B={B} H={H} N={N} d={d} rope={rope}")
    Q, K, V = wl.draw_tensors(9700 + N + d, (B, H, N, d), 0.5, "bf16")
    cs = wl.rope_tables_3d_factored(*grid, d)
    T = wl.expand_rope_tables(*cs) if rope != "none" else None
    O_ref, S_ref, z_ref = orc.bidirectional(Q, K, V, 1e-6, rope=T)
    Qd, Kd, Vd = _token_major(Q), _token_major(K), _token_major(V)
    dsc = sv.desc_of(Qd)
    dev = [torch.from_numpy(np.ascontiguousarray(t)).cuda() for t in cs]
    arg = {"none": (), "table": (torch.from_numpy(T).cuda() if T is not None else None,),
           "axes": (sv.Rope3D.from_tensors(*dev),)}[rope]
    sfx = {"none": "", "table": "_rope", "axes": "_rope3d"}[rope]
    ws = new_workspace(B, H, N, d)
    for form in ("layer", "block"):
        S, z = new_state(B, H, d)
        O = torch.full_like(Qd, float("nan"))
        assert O.stride() == Qd.stride()
        if form == "layer":
            getattr(sv, "sv_linattn_state" + sfx)(Kd, Vd, dsc, *arg, 0, N, 0, S, z, ws)
            getattr(sv, "sv_linattn_apply" + sfx)(Qd, dsc, *arg, 0, N, S, z, 1e-6, O)
        else:
            getattr(sv, "sv_block_linattn_step" + sfx)(Qd, Kd, Vd, dsc, *arg, S, z, 1e-6, O, ws)
        torch.cuda.synchronize()
        # rotated keys are rounded to bf16 once more: a relative error of 2^-9 / sqrt(3) per term
        assert metrics.rel_l2(to_host(S), S_ref) <= (1e-5 if rope == "none" else 3e-3)
        assert metrics.rel_l2(to_host(z), z_ref) <= 1e-5
        metrics.check(to_host(O), O_ref, "bf16", f"O ({form})")
