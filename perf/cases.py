"""The timed workloads: what a sequence-parallel Llama training step has one GPU do.

Each case is one pass through the public binding as a training program calls it, on the
head shards of the models the framework is made for (P = 8 unless a case says otherwise):

  attn      attention of one layer on attention-side tensors, forward (the rematerialised
            forward under activation checkpointing) or forward and backward
  step      the whole attention part of a layer on sequence-side tensors: re-layouts, forward,
            backward; either with separate re-layouts or folded into the attention kernels
  varlen    packed documents, forward and backward
  ring      one device of a ring schedule: its diagonal block and one block from the past,
            forward, merge and both blocks' backward
  relayout  one tensor packed and unpacked
  pointwise the operators between the matrix products of one layer, forward and backward
"""
from __future__ import annotations

import math
import random

import torch

import paper_2604_27089_amd.binding as sp

# Head shards of one GPU: (query heads, key/value heads, head dim) per model at P = 8 (the tiny one at P = 4).
SHARDS = {
    "tiny": (2, 1, 64),
    "1b": (4, 1, 64),
    "3b": (3, 1, 128),
    "8b": (4, 1, 128),
    "70b": (8, 1, 128),
    "13b": (5, 5, 128),
}
# Llama layer widths outside attention: (model dim, heads, head dim, feed-forward dim).
LAYERS = {
    "1b": (2048, 32, 64, 8192),
    "3b": (3072, 24, 128, 8192),
    "8b": (4096, 32, 128, 14336),
    "13b": (5120, 40, 128, 13824),
    "70b": (8192, 64, 128, 28672),
}


def listed():
    return [
        # the smallest configuration: launches and their latency
        {"name": "tiny_512", "kind": "attn", "shard": "tiny", "B": 1, "S": 512, "train": True},
        # one short sequence, the fine-tuning length of the evaluated models
        {"name": "8b_4k", "kind": "attn", "shard": "8b", "B": 1, "S": 4096, "train": True},
        # a length that is a multiple of nothing, the forward that checkpointing runs a second time
        {"name": "3b_10007_fwd", "kind": "attn", "shard": "3b", "B": 1, "S": 10007, "train": False},
        # head dim 64
        {"name": "1b_16k", "kind": "attn", "shard": "1b", "B": 1, "S": 16384, "train": True},
        # a batch of short sequences, the usual shape before long-context training
        {"name": "8b_16x4k", "kind": "attn", "shard": "8b", "B": 16, "S": 4096, "train": True},
        # 32K context, re-layout folded into the attention kernels
        {"name": "8b_32k_folded", "kind": "step", "shard": "8b", "S_l": 4096, "P": 8, "folded": True},
        # 128K context with separate re-layouts: the headline configuration
        {"name": "8b_128k", "kind": "step", "shard": "8b", "S_l": 16384, "P": 8, "folded": False},
        # packed documents of mixed length
        {"name": "varlen_64k", "kind": "varlen", "shard": "8b", "T": 65536, "mean": 4096, "docs": 0},
        # one device's share of a ring over 32K rows
        {"name": "ring_4k", "kind": "ring", "Hq": 32, "Hkv": 8, "D": 128, "S": 4096},
        # the 70B-shaped query shard around the all-to-all
        {"name": "relayout_70b", "kind": "relayout", "B": 1, "S_l": 16384, "h": 8, "D": 128, "P": 8, "bits": 16},
        # one 8B layer's pointwise operators at 128K context (16384 tokens per GPU)
        {"name": "pointwise_16k", "kind": "pointwise", "layer": "8b", "T": 16384},
        # and a small layer on a few odd tokens
        {"name": "pointwise_509", "kind": "pointwise", "layer": "1b", "T": 509},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "step", "varlen", "varlen", "ring", "relayout", "pointwise"])
    if kind == "attn":
        shard = rng.choice(sorted(SHARDS))
        Hq = SHARDS[shard][0]
        S = _log_int(rng, 64, int(131072 / math.sqrt(max(Hq, 4) / 4)))
        B = _log_int(rng, 1, max(1, min(64, 65536 // S)))
        return {"kind": kind, "shard": shard, "B": B, "S": S, "train": rng.random() < 0.7}
    if kind == "step":
        shard = rng.choice(["1b", "3b", "8b"])
        folded = rng.random() < 0.5
        P = rng.choice([2, 4, 8])
        S_l = 2 ** rng.randint(8, 13) if folded else _log_int(rng, 64, 8192)
        return {"kind": kind, "shard": shard, "S_l": S_l, "P": P, "folded": folded}
    if kind == "varlen":
        return {"kind": kind, "shard": rng.choice(["1b", "3b", "8b", "13b"]), "T": _log_int(rng, 512, 131072),
                "mean": _log_int(rng, 256, 8192), "docs": rng.randrange(1 << 20)}
    if kind == "ring":
        Hq, Hkv, D = rng.choice([(32, 8, 128), (24, 8, 128), (32, 8, 64)])
        return {"kind": kind, "Hq": Hq, "Hkv": Hkv, "D": D, "S": _log_int(rng, 256, 8192)}
    if kind == "relayout":
        return {"kind": kind, "B": rng.randint(1, 2), "S_l": _log_int(rng, 16, 16384), "h": rng.choice([1, 2, 3, 4, 5, 8]),
                "D": rng.choice([64, 128]), "P": rng.choice([2, 4, 8]), "bits": rng.choice([16, 16, 32])}
    return {"kind": kind, "layer": rng.choice(sorted(LAYERS)), "T": _log_int(rng, 32, 16384)}


def _doc_lengths(case):
    """Lognormal document lengths with the case's mean, clipped to [128, 32768], cut to fill T rows."""
    rng, T = random.Random(case["docs"]), case["T"]
    out, left = [], T
    while left > 0:
        n = int(min(max(rng.lognormvariate(math.log(case["mean"]) - 0.5, 1.0), 128), 32768, left))
        out.append(n)
        left -= n
    return out


# ---------------------------------------------------------------------------- inputs and the timed pass
def _normal(gen, *shape, scale=1.0):
    return (torch.randn(shape, generator=gen, device="cuda") * scale).to(torch.bfloat16)


def _inputs(case, seed):
    """The pass's inputs, a function of the case and the seed only."""
    g = torch.Generator(device="cuda").manual_seed(1000003 * seed + 17)
    kind = case["kind"]
    if kind == "attn":
        Hq, Hkv, D = SHARDS[case["shard"]]
        B, S = case["B"], case["S"]
        t = {"q": _normal(g, B, S, Hq, D), "k": _normal(g, B, S, Hkv, D), "v": _normal(g, B, S, Hkv, D)}
        if case["train"]:
            t["do"] = _normal(g, B, S, Hq, D)
        return t
    if kind == "step":
        Hq, Hkv, D = SHARDS[case["shard"]]
        S_l, P = case["S_l"], case["P"]
        return {"q": _normal(g, 1, S_l, P * Hq, D), "k": _normal(g, 1, S_l, P * Hkv, D),
                "v": _normal(g, 1, S_l, P * Hkv, D), "do": _normal(g, 1, S_l, P * Hq, D)}
    if kind == "varlen":
        Hq, Hkv, D = SHARDS[case["shard"]]
        T, cu = case["T"], [0]
        lengths = _doc_lengths(case)
        for n in lengths:
            cu.append(cu[-1] + n)
        return {"q": _normal(g, T, Hq, D), "k": _normal(g, T, Hkv, D), "v": _normal(g, T, Hkv, D),
                "do": _normal(g, T, Hq, D), "cu": torch.tensor(cu, dtype=torch.int32, device="cuda"),
                "longest": max(lengths)}
    if kind == "ring":
        Hq, Hkv, D, S = case["Hq"], case["Hkv"], case["D"], case["S"]
        return {"q": _normal(g, 1, S, Hq, D), "do": _normal(g, 1, S, Hq, D),
                "k": [_normal(g, 1, S, Hkv, D) for _ in range(2)], "v": [_normal(g, 1, S, Hkv, D) for _ in range(2)]}
    if kind == "relayout":
        x = torch.randn((case["B"], case["S_l"], case["P"] * case["h"], case["D"]), generator=g, device="cuda")
        return {"x": x if case["bits"] == 32 else x.to(torch.bfloat16)}
    C, H, D, F = LAYERS[case["layer"]]
    T = case["T"]
    inv = torch.exp(torch.arange(D // 2, device="cuda", dtype=torch.float64) * (-math.log(500000.0) / (D // 2)))
    angle = torch.arange(T, device="cuda", dtype=torch.float64)[:, None] * inv[None, :]
    return {"x": _normal(g, T, C), "w": _normal(g, C, scale=0.1) + 1.0, "dy": _normal(g, T, C),
            "q": _normal(g, T, H, D), "dq": _normal(g, T, H, D),
            "cos": torch.cos(angle).float(), "sin": torch.sin(angle).float(),
            "g": _normal(g, T, F), "u": _normal(g, T, F), "da": _normal(g, T, F)}


def prepare(case, seed):
    state = _inputs(case, seed)
    state["case"] = case
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "attn":
        q, k, v = state["q"], state["k"], state["v"]
        o, lse = sp.sp_attn_fwd(q, k, v)
        if not case["train"]:
            return {"o": o, "lse": lse}
        dq, dk, dv = sp.sp_attn_bwd(q, k, v, o, lse, state["do"])
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    if kind == "step":
        q, k, v, do, P = state["q"], state["k"], state["v"], state["do"], case["P"]
        if case["folded"]:
            o, lse = sp.sp_attn_fwd_seqlayout(q, k, v, P)
            dq, dk, dv = sp.sp_attn_bwd_seqlayout(q, k, v, o, lse, do, P)
            return {"o": o, "dq": dq, "dk": dk, "dv": dv}
        qh, kh, vh = (sp.sp_pack_seq_to_head(t, P) for t in (q, k, v))
        oh, lse = sp.sp_attn_fwd(qh, kh, vh)
        o = sp.sp_unpack_head_to_seq(oh, P)
        grads = sp.sp_attn_bwd(qh, kh, vh, oh, lse, sp.sp_pack_seq_to_head(do, P))
        dq, dk, dv = (sp.sp_unpack_head_to_seq(t, P) for t in grads)
        return {"o": o, "dq": dq, "dk": dk, "dv": dv}
    if kind == "varlen":
        q, k, v, cu, longest = state["q"], state["k"], state["v"], state["cu"], state["longest"]
        o, lse = sp.sp_attn_varlen_fwd(q, k, v, cu, longest)
        dq, dk, dv = sp.sp_attn_varlen_bwd(q, k, v, o, lse, state["do"], cu, longest)
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    if kind == "ring":
        q, do, S = state["q"], state["do"], case["S"]
        o_acc = torch.zeros(q.shape, dtype=torch.float32, device=q.device)
        lse = torch.full((1, case["Hq"], S), -math.inf, dtype=torch.float32, device=q.device)
        o = torch.empty_like(q)
        for i in range(2):  # the device's own keys, then those of its predecessor
            ob, lb = sp.sp_attn_block_fwd(q, state["k"][i], state["v"][i], S * i)
            sp.sp_attn_merge(o_acc, lse, ob, lb, o_out=o if i == 1 else None)
        out = {"o": o, "lse": lse}
        ws = torch.empty(sp.sp_attn_block_bwd_workspace_bytes(1, S, S, case["Hq"], case["Hkv"], case["D"]),
                         dtype=torch.uint8, device=q.device)
        for i in range(2):  # Delta is a property of the finished rows: computed with the first block only
            stages = sp.SP_BWD_STAGE_ALL if i == 0 else sp.SP_BWD_STAGE_DKDV | sp.SP_BWD_STAGE_DQ
            grads = sp.sp_attn_block_bwd(q, state["k"][i], state["v"][i], o, lse, do, S * i, workspace=ws, stages=stages)
            for name, t in zip(("dq", "dk", "dv"), grads):
                out[f"{name}{i}"] = t
        return out
    if kind == "relayout":
        y = sp.sp_pack_seq_to_head(state["x"], case["P"])
        return {"packed": y, "back": sp.sp_unpack_head_to_seq(y, case["P"])}
    y, rstd = sp.sp_rmsnorm_fwd(state["x"], state["w"], 1e-5)
    qr = sp.sp_rope(state["q"], state["cos"], state["sin"])
    act = sp.sp_swiglu_fwd(state["g"], state["u"])
    dg, du = sp.sp_swiglu_bwd(state["g"], state["u"], state["da"])
    dq = sp.sp_rope(state["dq"], state["cos"], state["sin"], conjugate=True)
    dx, dw = sp.sp_rmsnorm_bwd(state["x"], state["w"], rstd, state["dy"])
    return {"y": y, "rstd": rstd, "qr": qr, "act": act, "dg": dg, "du": du, "dq": dq, "dx": dx, "dw": dw}


# ---------------------------------------------------------------------------- what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind in ("attn", "step", "varlen"):
        Hq, Hkv, D = SHARDS[case["shard"]]
        if kind == "attn":
            rows, pairs, train = case["B"] * case["S"], case["B"] * case["S"] * (case["S"] + 1) // 2, case["train"]
        elif kind == "step":
            rows, train = case["S_l"] * case["P"], True
            pairs = rows * (rows + 1) // 2
        else:
            rows, train = case["T"], True
            pairs = sum(n * (n + 1) // 2 for n in _doc_lengths(case))
        qb, kb = 2 * rows * Hq * D, 2 * rows * Hkv * D
        # q, k, v in, o out; training: do in, dq, dk, dv out
        return {"bytes": (4 * qb + 4 * kb) if train else (2 * qb + 2 * kb), "flops": (14 if train else 4) * D * Hq * pairs}
    if kind == "ring":
        Hq, Hkv, D, S = case["Hq"], case["Hkv"], case["D"], case["S"]
        pairs = S * (S + 1) // 2 + S * S
        qb, kb = 2 * S * Hq * D, 2 * S * Hkv * D
        return {"bytes": 5 * qb + 8 * kb, "flops": 14 * D * Hq * pairs}  # q, do in, o and two dq out; two k, v in, two dk, dv out
    if kind == "relayout":
        n = case["B"] * case["S_l"] * case["P"] * case["h"] * case["D"] * case["bits"] // 8
        return {"bytes": 4 * n, "flops": 0}  # each way: read and write
    C, H, D, F = LAYERS[case["layer"]]
    T = case["T"]
    # norm: x, y, then x, dy, dx; rotation: in and out, twice; gate: g, u, y, then g, u, dy, dg, du; both tables
    return {"bytes": 2 * T * (5 * C + 4 * H * D + 8 * F) + 2 * 4 * T * D, "flops": 0}


def tolerance(case):
    if case["kind"] == "relayout":
        return "exact"
    # bf16 results; the gradients of two correct orders of summation differ by up to 2.5e-3
    return {"rel": 1e-2}


# ---------------------------------------------------------------------------- the same outputs in 64 bits
def _softmax_rows(qc, k, vis, scale):
    s = (qc @ k.t()) * scale
    s.masked_fill_(~vis, -math.inf)
    lse = torch.logsumexp(s, dim=1, keepdim=True)
    return s, lse


def _attn_one(q, k, v, do, lo, hi, lse_final=None, o_final=None):
    """One head in 64 bits: q, do [S, D], k, v [N, D]; row i sees keys lo[i] .. hi[i]-1 (hi ascending)."""
    S, D = q.shape
    scale = 1.0 / math.sqrt(D)
    o, lse = torch.empty_like(q), torch.empty(S, dtype=q.dtype, device=q.device)
    grads = None if do is None else (torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v))
    step = 2048
    for a in range(0, S, step):
        b = min(S, a + step)
        j0, j1 = int(lo[a]), int(hi[b - 1])
        idx = torch.arange(j0, j1, device=q.device)
        vis = (idx[None, :] >= lo[a:b, None]) & (idx[None, :] < hi[a:b, None])
        kk, vv = k[j0:j1], v[j0:j1]
        s, ls = _softmax_rows(q[a:b], kk, vis, scale)
        if lse_final is not None:
            ls = lse_final[a:b, None]
        p = s.sub_(ls).exp_()
        o[a:b] = p @ vv
        lse[a:b] = ls[:, 0]
        if do is not None:
            rows = o[a:b] if o_final is None else o_final[a:b]
            delta = (do[a:b] * rows).sum(dim=1, keepdim=True)
            grads[2][j0:j1] += p.t() @ do[a:b]
            ds = (do[a:b] @ vv.t()).sub_(delta).mul_(p).mul_(scale)
            grads[0][a:b] = ds @ kk
            grads[1][j0:j1] += ds.t() @ q[a:b]
    return o, lse, grads


def _attn_heads(q, k, v, do, lo, hi):
    """q, do [S, Hq, D], k, v [N, Hkv, D] -> o, lse [Hq, S], (dq, dk, dv), all 64 bits."""
    G = q.shape[1] // k.shape[1]
    q, k, v = q.double(), k.double(), v.double()
    do = None if do is None else do.double()
    o, lse = torch.empty_like(q), torch.empty((q.shape[1], q.shape[0]), dtype=q.dtype, device=q.device)
    grads = None if do is None else (torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v))
    for h in range(q.shape[1]):
        kc, vc = k[:, h // G].contiguous(), v[:, h // G].contiguous()
        oh, lse[h], gh = _attn_one(q[:, h].contiguous(), kc, vc, None if do is None else do[:, h].contiguous(), lo, hi)
        o[:, h] = oh
        if do is not None:
            grads[0][:, h] = gh[0]
            grads[1][:, h // G] += gh[1]
            grads[2][:, h // G] += gh[2]
    return o, lse, grads


def _to_heads(x, P):
    _, S_l, H, D = x.shape
    return x.view(S_l, P, H // P, D).transpose(0, 1).reshape(P * S_l, H // P, D)


def _to_seq(y, P):
    S, h, D = y.shape
    return y.view(P, S // P, h, D).transpose(0, 1).reshape(1, S // P, P * h, D)


def exact(case, seed):
    kind = case["kind"]
    t = _inputs(case, seed)
    dev = "cuda"
    if kind == "attn":
        S = case["S"]
        lo, hi = torch.zeros(S, dtype=torch.int64, device=dev), torch.arange(1, S + 1, device=dev)
        outs = [_attn_heads(t["q"][b], t["k"][b], t["v"][b], t["do"][b] if case["train"] else None, lo, hi)
                for b in range(case["B"])]
        res = {"o": torch.stack([x[0] for x in outs]), "lse": torch.stack([x[1] for x in outs])}
        if case["train"]:
            for i, name in enumerate(("dq", "dk", "dv")):
                res[name] = torch.stack([x[2][i] for x in outs])
        return res
    if kind == "step":
        P, S = case["P"], case["S_l"] * case["P"]
        lo, hi = torch.zeros(S, dtype=torch.int64, device=dev), torch.arange(1, S + 1, device=dev)
        o, _, g = _attn_heads(*(_to_heads(t[n], P) for n in ("q", "k", "v", "do")), lo, hi)
        return {"o": _to_seq(o, P), "dq": _to_seq(g[0], P), "dk": _to_seq(g[1], P), "dv": _to_seq(g[2], P)}
    if kind == "varlen":
        cu = t["cu"].long()
        idx = torch.arange(case["T"], device=dev)
        lo = cu[torch.searchsorted(cu, idx, right=True) - 1]
        o, lse, g = _attn_heads(t["q"], t["k"], t["v"], t["do"], lo, idx + 1)
        return {"o": o, "lse": lse, "dq": g[0], "dk": g[1], "dv": g[2]}
    if kind == "ring":
        S, G = case["S"], case["Hq"] // case["Hkv"]
        zero, diag = torch.zeros(S, dtype=torch.int64, device=dev), torch.arange(1, S + 1, device=dev)
        his = (diag, torch.full((S,), S, dtype=torch.int64, device=dev))
        q, do = t["q"][0].double(), t["do"][0].double()
        ks, vs = [x[0].double() for x in t["k"]], [x[0].double() for x in t["v"]]
        o, lse = torch.empty_like(q), torch.empty((1, case["Hq"], S), dtype=torch.float64, device=dev)
        res = {}
        for i in range(2):
            res[f"dq{i}"], res[f"dk{i}"], res[f"dv{i}"] = torch.empty_like(q), torch.zeros_like(ks[i]), torch.zeros_like(vs[i])
        for h in range(case["Hq"]):
            kv = [(ks[i][:, h // G].contiguous(), vs[i][:, h // G].contiguous()) for i in range(2)]
            qh, dh = q[:, h].contiguous(), do[:, h].contiguous()
            parts = [_attn_one(qh, *kv[i], None, zero, his[i]) for i in range(2)]
            total = torch.logaddexp(parts[0][1], parts[1][1])
            oh = sum(p[0] * torch.exp(p[1] - total)[:, None] for p in parts)
            o[:, h], lse[0, h] = oh, total
            for i in range(2):
                gh = _attn_one(qh, *kv[i], dh, zero, his[i], lse_final=total, o_final=oh)[2]
                res[f"dq{i}"][:, h] = gh[0]
                res[f"dk{i}"][:, h // G] += gh[1]
                res[f"dv{i}"][:, h // G] += gh[2]
        return {"o": o[None], "lse": lse, **{name: x[None] for name, x in res.items()}}
    if kind == "relayout":
        B, S_l, P, h, D = (case[n] for n in ("B", "S_l", "P", "h", "D"))
        y = t["x"].view(B, S_l, P, h, D).transpose(1, 2).reshape(B, P * S_l, h, D)
        return {"packed": y, "back": t["x"]}
    x, w, dy = t["x"].double(), t["w"].double(), t["dy"].double()
    r = torch.rsqrt((x * x).mean(dim=1, keepdim=True) + 1e-5)
    gx = dy * w
    res = {"y": x * r * w, "rstd": r[:, 0]}
    cos, sin = t["cos"].double()[:, None, :], t["sin"].double()[:, None, :]

    def turn(z, s):
        a, b = z.double().chunk(2, dim=2)
        return torch.cat([a * cos - b * s, b * cos + a * s], dim=2)

    res["qr"] = turn(t["q"], sin)
    g, u, da = t["g"].double(), t["u"].double(), t["da"].double()
    sg = torch.sigmoid(g)
    res["act"], res["dg"], res["du"] = g * sg * u, da * u * sg * (1 + g * (1 - sg)), da * g * sg
    res["dq"] = turn(t["dq"], -sin)
    res["dx"] = gx * r - x * r ** 3 * (gx * x).mean(dim=1, keepdim=True)
    res["dw"] = (dy * x * r).sum(dim=0)
    return res
