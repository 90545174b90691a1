"""GPU parity of the state update over the numbers of workgroups that share a head (256 compute units: 1 at 129 heads and
more, 2, 3, 4, 5, 8, 12): a workgroup alone stores the state itself, few contributors fold long slices, many short
ones.  Carried state in place, ragged token counts, layer and block step."""
import numpy as np
import pytest

import paper_2509_24695_amd as sv
import sv_workloads as wl
from oracle import linattn_oracle as orc
from sv_workloads import metrics
from tests.gpu_util import new_state, new_workspace, say, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("BH", [256, 160, 128, 85, 64, 51, 32, 20])
@pytest.mark.parametrize("dtype,d,rope", [("bf16", 64, "none"), ("bf16", 64, "axes"), ("bf16", 112, "none"), ("bf16", 112, "axes"),
                                          ("bf16", 112, "table"), ("bf16", 128, "none"), ("f32", 64, "none"), ("f32", 112, "axes")])
def test_contributors(dtype, d, rope, BH):
    import torch
    grid = (1, 23, 37)
    N = grid[1] * grid[2]
    say(f"contributors {dtype} d={d} rope={rope} BH={BH}")
    Q, K, V = wl.draw_tensors(9300 + BH + d, (1, BH, N, d), 0.5, dtype)
    rng = np.random.Generator(np.random.PCG64(77))
    S0 = rng.standard_normal((1, BH, d, d), dtype=np.float32)
    z0 = np.abs(rng.standard_normal((1, BH, d), dtype=np.float32)) * 10
    cs = wl.rope_tables_3d_factored(*grid, d)
    T = wl.expand_rope_tables(*cs) if rope != "none" else None
    Qd, Kd, Vd = to_dev(Q), to_dev(K), to_dev(V)
    dsc, ws = sv.desc_of(Qd), new_workspace(1, BH, N, d)
    dev = [torch.from_numpy(np.ascontiguousarray(t)).cuda() for t in cs]
    arg = {"none": (), "table": (torch.from_numpy(T).cuda() if T is not None else None,),
           "axes": (sv.Rope3D.from_tensors(*dev),)}[rope]
    sfx = {"none": "", "table": "_rope", "axes": "_rope3d"}[rope]
    s_tol = 1e-5 if rope == "none" or dtype == "f32" else 3e-3      # rotated bf16 keys: 2^-9 / sqrt(3) per term
    O_ref, S_ref, z_ref = orc.block_step(Q, K, V, S0.astype(np.float64), z0.astype(np.float64), 1e-6, rope=T)
    for form in ("state", "block", "lookahead"):
        S, z = new_state(1, BH, d)
        S.copy_(torch.from_numpy(S0))
        z.copy_(torch.from_numpy(z0))
        O = torch.full_like(Qd, float("nan"))
        if form == "state":
            getattr(sv, "sv_linattn_state" + sfx)(Kd, Vd, dsc, *arg, 0, N, 1, S, z, ws)
        else:
            step = "sv_block_linattn_step" if form == "block" else "sv_block_linattn_lookahead"
            getattr(sv, step + sfx)(Qd, Kd, Vd, dsc, *arg, S, z, 1e-6, O, ws)
        torch.cuda.synchronize()
        assert sv.sv_linattn_workspace_status(ws, 1, BH, d) == 0
        if form == "lookahead":
            assert np.array_equal(to_host(S), S0) and np.array_equal(to_host(z), z0)
        else:
            assert metrics.rel_l2(to_host(S), S_ref) <= s_tol and metrics.rel_l2(to_host(z), z_ref) <= 1e-5
        if form != "state":
            metrics.check(to_host(O), O_ref, dtype, f"O ({form})")
