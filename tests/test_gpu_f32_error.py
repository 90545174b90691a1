"""The fp32 mode's sums are no further from 64 bits than plain fp32 sums in short chunks: one fused multiply-add per token in
token order inside a chunk of 32 tokens and more, about 512 chunks over all heads (at most 32 per head), the chunks
added in order.  Tolerances for parity (1e-5) are far wider and do not see a summation order that loses half a digit."""
import numpy as np
import pytest

import paper_2509_24695_amd as sv
import sv_workloads as wl
from tests.gpu_util import new_state, new_workspace, say, to_dev, to_host

pytestmark = pytest.mark.gpu


def _chunked_fp32(fk, v, BH):
    """(S, z) of heads [h][N][d] in fp32 by chunks; products exact (the 64-bit product and sum are rounded once)."""
    heads, N, d = fk.shape
    tiles = (N + 31) // 32
    C = max(1, min(512 // BH, 32, tiles))
    S, z = np.zeros((heads, d, d), np.float32), np.zeros((heads, d), np.float32)
    for c in range(C):
        Sc, zc = np.zeros_like(S), np.zeros_like(z)
        for t in range(c * tiles // C * 32, min((c + 1) * tiles // C * 32, N)):
            Sc = (Sc + fk[:, t, :, None].astype(np.float64) * v[:, t, None, :]).astype(np.float32)
            zc = zc + fk[:, t]
        S, z = S + Sc, z + zc
    return S, z


def _rms(a, ref):
    return float(np.sqrt(((a.astype(np.float64) - ref) ** 2).sum() / (ref ** 2).sum()))


@pytest.mark.parametrize("d,BH,N", [(32, 2, 1024), (32, 20, 384), (32, 2, 1153), (32, 33, 769), (64, 2, 256), (64, 33, 193), (64, 2, 2000),
                                    (64, 160, 384), (112, 8, 384),
                                    (112, 160, 384), (128, 32, 1024), (112, 64, 128), (128, 128, 128)])
def test_sums_are_as_exact_as_short_chunks(d, BH, N):
    import torch
    say(f"f32_error d={d} BH={BH} N={N}")
    _, K, V = wl.draw_tensors(9500 + N + d, (1, BH, N, d), 0.5, "f32")
    Kd, Vd = to_dev(K), to_dev(V)
    S, z = new_state(1, BH, d)
    sv.sv_linattn_state(Kd, Vd, sv.desc_of(Kd), 0, N, 0, S, z, new_workspace(1, BH, N, d))
    torch.cuda.synchronize()
    heads = min(BH, 8)
    fk, v = np.maximum(K[0, :heads], 0), V[0, :heads]
    S64 = np.matmul(fk.astype(np.float64).transpose(0, 2, 1), v.astype(np.float64))
    z64 = fk.astype(np.float64).sum(1)
    S32, z32 = _chunked_fp32(fk, v, BH)
    for name, got, plain, ref in (("S", to_host(S)[0, :heads], S32, S64), ("z", to_host(z)[0, :heads], z32, z64)):
        # both are the root mean square of ref.size rounding errors: each known to a share of 1 / sqrt(2 size); three of those
        slack = 1 + 3 / np.sqrt(ref.size)
        print(f"{name}: {_rms(got, ref):.3e}, in chunks {_rms(plain, ref):.3e}, at most x {slack:.3f}", flush=True)
        assert _rms(got, ref) <= slack * _rms(plain, ref)
