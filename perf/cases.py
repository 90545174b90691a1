"""The calls whose speed counts: what a program that generates video with this library asks of it, pass by pass.

Three kinds of pass, all through the C ABI's binding:

  layer    one bidirectional attention layer: sv_linattn_state over all tokens, then sv_linattn_apply
  stream   block-causal generation from an empty state: for every block `noisy` denoising passes that leave the
           carried state alone (sv_block_linattn_lookahead) and one that commits it (sv_block_linattn_step)
  tconv    the Mix-FFN's temporal convolution over consecutive blocks of frames, each again with `noisy` passes that
           leave the conv cache alone and one that replaces it (one block: the whole clip, no cache)

with the options that programs use: the rotation (none, a full table, per-axis tables), the layout of the token
tensors ("bhnd": heads outside tokens, "bnhd": a projection's output as it lies in memory), the four head dimensions,
bf16 and fp32.  Values are what the benchmark uses: 0.5 * N(0, 1) tokens, N(0, 1) frames with weights of variance
1 / (3 D).
"""
from __future__ import annotations

import math

import torch

import paper_2509_24695_amd as sv
import sv_workloads as wl

EPS = 1e-6


def _attn(name, kind, B, H, grid, d, dtype="bf16", rope="none", layout="bhnd", blocks=1, noisy=0):
    frames, rows, cols = grid
    return {"name": name, "kind": kind, "B": B, "H": H, "frames": frames, "rows": rows, "cols": cols, "d": d,
            "dtype": dtype, "rope": rope, "layout": layout, "blocks": blocks, "noisy": noisy}


def _tconv(name, B, T, HW, D, blocks=1, noisy=0):
    return {"name": name, "kind": "tconv", "B": B, "T": T, "HW": HW, "D": D, "blocks": blocks, "noisy": noisy}


def listed():
    return [
        # the benchmark's layer: a 720p clip, conditional and unconditional half of the guidance in one call
        _attn("clip_720p_pair", "layer", 2, 32, (21, 45, 80), 64),
        # the 2B model's heads on a 480p clip, guidance pair, rotation by per-axis tables, tensors as the q/k/v
        # projections leave them
        _attn("clip_480p_model", "layer", 2, 20, (21, 30, 52), 112, rope="axes", layout="bnhd"),
        # the same heads for a program that keeps one rotation table for the whole clip
        _attn("clip_480p_table", "layer", 1, 20, (21, 30, 52), 112, rope="table"),
        # single images as one-frame clips in a batch, narrow heads
        _attn("image_d32", "layer", 4, 32, (1, 64, 64), 32),
        # fp32 twin of a block of tokens, to check a bf16 pipeline against
        _attn("check_f32", "layer", 1, 32, (3, 30, 52), 64, dtype="f32"),
        # the smallest call of the test and benchmark set, fp32: launches and latency
        _attn("tiny_f32", "layer", 1, 2, (4, 16, 16), 32, dtype="f32"),
        # the benchmark's block stream at 480p: ten blocks of three latent frames
        _attn("stream_480p", "stream", 1, 32, (3, 30, 52), 64, blocks=10),
        # the 720p block stream with rotation
        _attn("stream_720p_axes", "stream", 1, 32, (3, 45, 80), 64, rope="axes", blocks=4),
        # few-step generation with the 2B model's heads: three noisy passes per block, then the clean one
        _attn("denoise_480p_model", "stream", 1, 20, (3, 30, 52), 112, rope="axes", blocks=2, noisy=3),
        # a server's batch of sequences that advance frame by frame, wide heads
        _attn("serve_batch_d128", "stream", 8, 20, (1, 30, 52), 128, blocks=3, noisy=1),
        # temporal convolution of the bidirectional model: the whole 480p clip
        _tconv("tconv_clip_480p", 1, 21, 30 * 52, 2240),
        # and of the block-causal one: blocks of three frames with the cache carried on
        _tconv("tconv_stream_480p", 1, 3, 30 * 52, 2240, blocks=3, noisy=1),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """Another case of the same ranges: grids from a thumbnail to 720p, any number of frames up to the clip's 21, odd
    and ragged sizes, every option."""
    kind = rng.choice(["layer", "layer", "stream", "stream", "tconv"])
    while True:
        if kind == "tconv":
            c = _tconv("", rng.choice([1, 1, 2]), rng.choice([1, 2, 3, 3, 5, 21]), _log_int(rng, 40, 3600),
                       8 * _log_int(rng, 8, 280), rng.choice([1, 2, 3]), rng.choice([0, 1]))
        else:
            dtype = rng.choice(["bf16", "bf16", "bf16", "bf16", "f32"])
            d = rng.choice([64, 64, 64, 112, 112, 112, 128, 32])
            grid = (rng.choice([1, 2, 3, 3, 3, 5, 21] if kind == "stream" else [1, 4, 9, 13, 21, 21]),
                    _log_int(rng, 8, 45), _log_int(rng, 9, 80))
            c = _attn("", kind, rng.choice([1, 1, 2, 2, 3, 4, 8]), rng.choice([2, 5, 8, 16, 20, 20, 32, 32]), grid, d,
                      dtype, rng.choice(["none", "axes", "axes", "table"]), rng.choice(["bhnd", "bhnd", "bnhd"]),
                      rng.choice([2, 3, 4]) if kind == "stream" else 1, rng.choice([0, 1, 3]) if kind == "stream" else 0)
        del c["name"]
        w = work(c)
        slow = c.get("dtype") == "f32" or c.get("d") == 32           # no case of these as large as the bf16 clips
        if w["bytes"] <= (0.4e9 if slow else 2.4e9) and w["flops"] <= (2e10 if slow else 9e11):
            return c


# ---- inputs -------------------------------------------------------------------------------------------------------

def _tokens(case, gen):
    B, H, N, d = case["B"], case["H"], case["frames"] * case["rows"] * case["cols"], case["d"]
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    shape = (B, H, N, d) if case["layout"] == "bhnd" else (B, N, H, d)
    x = (torch.randn(shape, generator=gen, device="cuda") * 0.5).to(dt)
    return x if case["layout"] == "bhnd" else x.permute(0, 2, 1, 3)


def _rope_of_block(case, m):
    """Rotation tables of block m (the time axis goes on from block to block)."""
    f, r, c, d = case["frames"], case["rows"], case["cols"], case["d"]
    axes = [torch.from_numpy(t).cuda() for t in wl.rope_tables_3d_factored(f, r, c, d, t0=m * f)]
    table = torch.from_numpy(wl.rope_table_3d(f, r, c, d, t0=m * f)).cuda() if case["rope"] == "table" else None
    return {"axes": axes, "table": table, "r3": sv.Rope3D.from_tensors(*axes)}


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    if case["kind"] == "tconv":
        B, T, HW, D = (case[k] for k in ("B", "T", "HW", "D"))
        passes = case["blocks"] * (case["noisy"] + 1)
        W = (torch.randn((3, D, D), generator=gen, device="cuda") / math.sqrt(3 * D)).to(torch.bfloat16)
        x = [torch.randn((B, T, HW, D), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(passes)]
        cache = torch.empty((B, HW, D), dtype=torch.bfloat16, device="cuda") if case["blocks"] > 1 else None
        return {"case": case, "W": W, "x": x, "y": [torch.empty_like(t) for t in x], "cache": cache}
    B, H, N, d = case["B"], case["H"], case["frames"] * case["rows"] * case["cols"], case["d"]
    passes = case["blocks"] * (case["noisy"] + 1)
    qkv = [tuple(_tokens(case, gen) for _ in range(3)) for _ in range(passes)]
    rope = [_rope_of_block(case, m) for m in range(case["blocks"])] if case["rope"] != "none" else None
    return {"case": case, "qkv": qkv, "O": [torch.empty_like(q) for q, _, _ in qkv], "desc": sv.desc_of(qkv[0][0]), "rope": rope,
            "S": torch.empty((B, H, d, d), device="cuda"), "z": torch.empty((B, H, d), device="cuda"),
            "ws": torch.empty(sv.sv_linattn_workspace_bytes(B, H, N, d), dtype=torch.uint8, device="cuda")}


# ---- one pass -------------------------------------------------------------------------------------------------------

def _run_layer(s):
    stream = torch.cuda.current_stream()
    (q, k, v), O, dsc, S, z, ws, mode = s["qkv"][0], s["O"][0], s["desc"], s["S"], s["z"], s["ws"], s["case"]["rope"]
    N = dsc.N
    if mode == "none":
        sv.sv_linattn_state(k, v, dsc, 0, N, 0, S, z, ws, stream=stream)
        sv.sv_linattn_apply(q, dsc, 0, N, S, z, EPS, O, stream=stream)
    elif mode == "table":
        t = s["rope"][0]["table"]
        sv.sv_linattn_state_rope(k, v, dsc, t, 0, N, 0, S, z, ws, stream=stream)
        sv.sv_linattn_apply_rope(q, dsc, t, 0, N, S, z, EPS, O, stream=stream)
    else:
        r3 = s["rope"][0]["r3"]
        sv.sv_linattn_state_rope3d(k, v, dsc, r3, 0, N, 0, S, z, ws, stream=stream)
        sv.sv_linattn_apply_rope3d(q, dsc, r3, 0, N, S, z, EPS, O, stream=stream)
    return {"O": O, "S": S, "z": z}


def _run_stream(s):
    stream = torch.cuda.current_stream()
    case, dsc, S, z, ws = s["case"], s["desc"], s["S"], s["z"], s["ws"]
    mode, per_block = case["rope"], case["noisy"] + 1
    S.zero_()
    z.zero_()
    for i, ((q, k, v), O) in enumerate(zip(s["qkv"], s["O"])):
        m, commit = i // per_block, i % per_block == per_block - 1
        if mode == "none":
            (sv.sv_block_linattn_step if commit else sv.sv_block_linattn_lookahead)(
                q, k, v, dsc, S, z, EPS, O, ws, stream=stream)
        elif mode == "table":
            (sv.sv_block_linattn_step_rope if commit else sv.sv_block_linattn_lookahead_rope)(
                q, k, v, dsc, s["rope"][m]["table"], S, z, EPS, O, ws, stream=stream)
        else:
            (sv.sv_block_linattn_step_rope3d if commit else sv.sv_block_linattn_lookahead_rope3d)(
                q, k, v, dsc, s["rope"][m]["r3"], S, z, EPS, O, ws, stream=stream)
    return {"O": s["O"], "S": S, "z": z}


def _run_tconv(s):
    stream = torch.cuda.current_stream()
    case, W, cache = s["case"], s["W"], s["cache"]
    B, T, HW, D, per_block = case["B"], case["T"], case["HW"], case["D"], case["noisy"] + 1
    for i, (x, y) in enumerate(zip(s["x"], s["y"])):
        m, commit = i // per_block, i % per_block == per_block - 1
        sv.sv_tconv_block_step(x, W, cache if m > 0 else None, y, cache if commit else None, B, T, HW, D, stream=stream)
    return {"y": s["y"], "cache": cache} if cache is not None else {"y": s["y"]}


def run(state):
    return {"layer": _run_layer, "stream": _run_stream, "tconv": _run_tconv}[state["case"]["kind"]](state)


# ---- what a pass cannot do without ------------------------------------------------------------------------------------

def work(case):
    passes, blocks = case["blocks"] * (case["noisy"] + 1), case["blocks"]
    if case["kind"] == "tconv":
        B, T, HW, D = (case[k] for k in ("B", "T", "HW", "D"))
        tokens, cache = B * T * HW * D, B * HW * D
        carried = passes - (case["noisy"] + 1)                       # passes of all blocks but the first read a cache
        bytes_ = 2 * (passes * (2 * tokens + 3 * D * D) + carried * cache + (blocks * cache if blocks > 1 else 0))
        # the frame behind a block is zero, and so is the one in front of the first block: their taps are no work
        taps = passes * (3 * T - 2) + carried
        return {"bytes": bytes_, "flops": 2 * D * D * B * HW * taps}
    B, H, N, d = case["B"], case["H"], case["frames"] * case["rows"] * case["cols"], case["d"]
    elem = 4 if case["dtype"] == "f32" else 2
    state = B * H * (d * d + d) * 4
    half = d // 2
    table = {"none": 0, "table": N * half * 8,
             "axes": (case["frames"] * (half - 2 * (3 * half // 8)) + (case["rows"] + case["cols"]) * (3 * half // 8)) * 8}[case["rope"]]
    moved = state * (passes + blocks) if case["kind"] == "stream" else state
    return {"bytes": passes * (4 * B * H * N * d * elem + table) + moved, "flops": passes * B * H * N * (4 * d * d + 4 * d)}


def tolerance(case):
    """fp32: sums of products in another order.  bf16: one rounding of the outputs (1.7e-3 in the 2-norm) and, with a
    rotation, one of the rotated features (2.0e-3 with both).  Four times what the calls measure against 64-bit results."""
    if case.get("dtype") == "f32":
        return {"rel": 2e-6, "max": 2e-5}
    return {"rel": 8e-3, "max": 2e-2}


# ---- the same in 64 bits ------------------------------------------------------------------------------------------------

def _rotated(x, table):
    if table is None:
        return x
    c, s = table[..., 0], table[..., 1]
    a, b = x[:, 0::2], x[:, 1::2]
    return torch.stack([a * c - b * s, a * s + b * c], dim=-1).reshape(x.shape)


def _table64(case, rope):
    if rope is None:
        return None
    t, r, c = (a.double() for a in rope["axes"])
    f, rows, cols = t.shape[0], r.shape[0], c.shape[0]
    full = torch.cat([t[:, None, None].expand(f, rows, cols, *t.shape[1:]),
                      r[None, :, None].expand(f, rows, cols, *r.shape[1:]),
                      c[None, None, :].expand(f, rows, cols, *c.shape[1:])], dim=3)
    return full.reshape(f * rows * cols, case["d"] // 2, 2)


def _exact_tconv(s):
    case, W, cache, ys = s["case"], s["W"].double(), None, []
    per_block = case["noisy"] + 1
    for i, x in enumerate(s["x"]):
        x = x.double()
        front = torch.zeros_like(x[:, 0]) if cache is None else cache
        padded = torch.cat([front[:, None], x, torch.zeros_like(x[:, :1])], dim=1)
        y = x.clone()
        for tap in range(3):
            y += padded[:, tap:tap + case["T"]] @ W[tap].t().contiguous()
        ys.append(y)
        if i % per_block == per_block - 1:
            cache = x[:, -1].clone()
    return {"y": ys, "cache": cache} if s["cache"] is not None else {"y": ys}


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "tconv":
        return _exact_tconv(s)
    B, H, d, per_block = case["B"], case["H"], case["d"], case["noisy"] + 1
    S = torch.zeros((B, H, d, d), dtype=torch.float64, device="cuda")
    z = torch.zeros((B, H, d), dtype=torch.float64, device="cuda")
    outs = []
    for i, (q, k, v) in enumerate(s["qkv"]):
        table = _table64(case, s["rope"][i // per_block]) if s["rope"] is not None else None
        O = torch.empty(q.shape, dtype=torch.float64, device="cuda")
        commit = case["kind"] == "layer" or i % per_block == per_block - 1
        for b in range(B):
            for h in range(H):
                fk, fq = (t[b, h].double().clamp_min(0) for t in (k, q))
                S1 = S[b, h] + _rotated(fk, table).t().contiguous() @ v[b, h].double()
                z1 = z[b, h] + fk.sum(0)
                O[b, h] = (_rotated(fq, table) @ S1) / (fq @ z1 + EPS)[:, None]
                if commit:
                    S[b, h], z[b, h] = S1, z1
        outs.append(O)
    return {"O": outs[0] if case["kind"] == "layer" else outs, "S": S, "z": z}
