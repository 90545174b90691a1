"""Heads of few tokens in the fp32-arithmetic state kernel: four workgroups with a quarter of the state each while four per head fit on the device's 256
compute units (64 heads), one beyond; and the state in three bf16 pieces in the apply kernel of bf16 tokens at d = 32, which has to be as good
as fp32 products for any state, infinities among it."""
import numpy as np
import pytest

import paper_2509_24695_amd as sv
import sv_workloads as wl
from oracle import linattn_oracle as orc
from sv_workloads import metrics
from tests.gpu_util import new_state, new_workspace, say, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rope", ["none", "table", "axes"])
@pytest.mark.parametrize("dtype,d,B,H,grid,layout", [
    ("f32", 32, 1, 1, (1, 1, 1), "bhnd"), ("f32", 32, 1, 7, (1, 3, 11), "bhnd"), ("f32", 32, 2, 4, (1, 17, 31), "bnhd"), ("f32", 32, 2, 32, (1, 16, 31), "bhnd"),
    ("f32", 32, 5, 13, (1, 16, 31), "bhnd"), ("bf16", 32, 1, 9, (1, 5, 13), "bnhd"), ("bf16", 32, 2, 32, (1, 1, 513), "bhnd"), ("bf16", 32, 1, 65, (1, 7, 9), "bhnd"),
    ("f32", 64, 1, 1, (1, 1, 7), "bhnd"), ("f32", 64, 1, 9, (1, 5, 13), "bnhd"), ("f32", 64, 2, 32, (1, 10, 19), "bhnd"), ("f32", 64, 1, 65, (1, 10, 19), "bhnd")])
def test_quarters_of_the_state(dtype, d, B, H, grid, layout, rope):
    import torch
    N = grid[0] * grid[1] * grid[2]
    say(f"f32_quarters {dtype} d={d} B={B} H={H} grid={grid} {layout} {rope}")
    _, K, V = wl.draw_tensors(9950 + N + d, (B, H, N, d), 0.5, dtype)
    rng = np.random.Generator(np.random.PCG64(95))
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
    S_ref, z_ref = orc.state(K, V, rope=T if rope != "none" else None)
    for accumulate, S_want, z_want in ((1, S0 + S_ref, z0 + z_ref), (0, S_ref, z_ref)):
        state(Kd, Vd, dsc, *arg, 0, N, accumulate, S, z, ws)
        torch.cuda.synchronize()
        assert metrics.rel_l2(to_host(S), S_want) <= 1e-5 and metrics.rel_l2(to_host(z), z_want) <= 1e-5     # fp32 sums


@pytest.mark.parametrize("layout", ["bhnd", "bnhd"])
@pytest.mark.parametrize("rope", ["none", "axes"])
@pytest.mark.parametrize("dtype,d,N", [("f32", 32, (640, 512)), ("bf16", 32, (896, 640)), ("f32", 64, (191, 192))])
def test_quarters_give_the_bits_of_one_workgroup(dtype, d, N, rope, layout):
    """64 heads are summed by quarters, 65 and 66 by one workgroup each; waves with several tiles, whose order is the head's (token-major: the batch's)."""
    import torch
    n, B, most = N[rope != "none"], *((1, 65) if layout == "bhnd" else (2, 33))
    say(f"f32_quarters bits {dtype} d={d} {rope} {layout}")
    _, K, V = wl.draw_tensors(9960 + d, (B, most, n, d), 0.5, dtype)
    Kd, Vd = to_dev(K), to_dev(V)
    keep = [torch.from_numpy(np.ascontiguousarray(t)).cuda() for t in wl.rope_tables_3d_factored(1, n // 16, 16, d)] if rope != "none" else []
    got = []
    for H in (most, most - 1):
        k, v = Kd[:, :H].contiguous(), Vd[:, :H].contiguous()
        if layout == "bnhd":
            k, v = (x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for x in (k, v))
        S, z = new_state(B, H, d)
        call = sv.sv_linattn_state if rope == "none" else sv.sv_linattn_state_rope3d
        call(k, v, sv.desc_of(k), *([] if rope == "none" else [sv.Rope3D.from_tensors(*keep)]), 0, n, 0, S, z, new_workspace(B, H, n, d))
        torch.cuda.synchronize()
        got.append((S[:, :most - 1], z[:, :most - 1]))
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("N", [1, 15, 16, 17, 67])
def test_state_in_three_pieces(N):
    """State entries of 24 significant bits over forty orders of magnitude down to 1e-20: every output within its own rounding to bf16 (2^-8 of it, and the
    rounding of sums that cancel: 2^-20 of the sum of magnitudes).  One infinite entry: as in fp32."""
    import torch
    B, H, d = 1, 3, 32
    say(f"f32 pieces N={N}")
    Q, _, _ = wl.draw_tensors(9970 + N, (B, H, N, d), 0.5, "bf16")
    rng = np.random.Generator(np.random.PCG64(96))
    S0 = rng.standard_normal((B, H, d, d), dtype=np.float32) * (10.0 ** rng.uniform(-20, 20, (B, H, 1, d))).astype(np.float32)
    z0 = np.abs(rng.standard_normal((B, H, d), dtype=np.float32)) + 0.5
    Qd = to_dev(Q)
    S, z = new_state(B, H, d)
    z.copy_(torch.from_numpy(z0))
    q = np.maximum(to_host(Qd).astype(np.float64), 0.0)
    den = np.einsum("bhnk,bhk->bhn", q, z0.astype(np.float64))[..., None] + 1e-6
    for bad in (False, True):
        S_now = S0.copy()
        if bad:
            S_now[:, :, 5, 7] = np.inf
        S.copy_(torch.from_numpy(S_now))
        O = torch.full_like(Qd, 3.0)
        sv.sv_linattn_apply(Qd, sv.desc_of(Qd), 0, N, S, z, 1e-6, O)
        torch.cuda.synchronize()
        got = to_host(O).astype(np.float64)
        want, size = np.matmul(q, S0.astype(np.float64)) / den, np.matmul(q, np.abs(S0).astype(np.float64)) / den
        ok = np.abs(got - want) <= 2.0 ** -8 * np.abs(want) + 2.0 ** -20 * size
        if bad:
            positive = q[:, :, :, 5] > 0                       # inf * q, and NaN where q is 0
            assert np.isposinf(got[:, :, :, 7][positive]).all() and np.isnan(got[:, :, :, 7][~positive]).all()
            ok[:, :, :, 7] = True
        assert ok.all()


# sizes (powers of two) of the queries, the state and the key sums; eps = 0
@pytest.mark.parametrize("rope", ["none", "axes"])
@pytest.mark.parametrize("q2,s2,z2", [(0, -127, -127), (0, -121, -121), (0, -113, -113), (0, -110, -110), (0, -20, -136), (0, -20, -131), (0, 100, 121), (-130, 0, 0),
                                      (-130, 0, -6), (-60, -60, -60), (-64, -64, -64), (0, 0, 0)])
def test_small_states_and_denominators(q2, s2, z2, rope):
    """bf16, d = 32: the quotients, where a reciprocal of the denominator is infinite or its state's bf16 pieces are below the normal numbers: within
    the rounding to bf16 and that of sums and products to multiples of 2^-149 (2^-16 of the sum of magnitudes); rotated features: five times that.
    A column of zeros stays zero."""
    import torch
    B, H, N, d = 1, 3, 70, 32
    say(f"f32 small states {q2} {s2} {z2} {rope}")
    rng = np.random.Generator(np.random.PCG64(97))
    Qd = torch.from_numpy(np.ldexp(np.abs(rng.standard_normal((B, H, N, d))) + 0.25, q2).astype(np.float32)).cuda().bfloat16()
    S0 = np.ldexp(rng.standard_normal((B, H, d, d)), s2).astype(np.float32)
    S0[..., 5] = 0.0
    z0 = np.ldexp(np.abs(rng.standard_normal((B, H, d))) + 0.25, z2).astype(np.float32)
    S, z = new_state(B, H, d)
    S.copy_(torch.from_numpy(S0))
    z.copy_(torch.from_numpy(z0))
    cs = wl.rope_tables_3d_factored(1, 7, 10, d)
    keep = [torch.from_numpy(np.ascontiguousarray(t)).cuda() for t in cs]
    O = torch.full_like(Qd, float("nan"))
    if rope == "none":
        sv.sv_linattn_apply(Qd, sv.desc_of(Qd), 0, N, S, z, 0.0, O)
    else:
        sv.sv_linattn_apply_rope3d(Qd, sv.desc_of(Qd), sv.Rope3D.from_tensors(*keep), 0, N, S, z, 0.0, O)
    torch.cuda.synchronize()
    q, got = to_host(Qd).astype(np.float64), to_host(O).astype(np.float64)
    den = np.matmul(q, z0.astype(np.float64)[..., None])
    if rope != "none":
        T = wl.expand_rope_tables(*cs).astype(np.float64)                  # [N][d/2][2]
        a, b = q[..., 0::2], q[..., 1::2]
        q = np.stack([a * T[..., 0] - b * T[..., 1], a * T[..., 1] + b * T[..., 0]], -1).reshape(q.shape)
    want, size = np.matmul(q, S0.astype(np.float64)) / den, np.matmul(np.abs(q), np.abs(S0).astype(np.float64)) / den
    assert (np.abs(got - want) <= 2.0 ** -8 * np.abs(want) + (1 if rope == "none" else 5) * 2.0 ** -16 * size).all()
    assert (got[..., 5] == 0).all()
