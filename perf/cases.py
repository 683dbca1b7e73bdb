"""The work this framework is used for, as cases whose time is measured.

Four kinds, each through the package's public entry points:

  ring    one rank's share of Double-Ring-Attention over resident K/V chunks (`RingReplay`): the forward
          replay, the backward replay, or both (one attention of a training step)
  step    one attention step without a mask (`attn_step_fwd`, `attn_step_bwd`): every key visible to every
          row, query and key lengths of their own (a single context-parallel rank, cross attention)
  update  the log-sum-exp merge of two partial results (`lse_merge`)
  layout  the local work of head parallelism around the ring: heads packed into messages, received messages
          unpacked, K/V heads replicated (`permute_rows`), the replicas' gradients reduced (`reduce_replicas`)

Inputs are drawn on the GPU from the seed: activations N(0,1) * sigma rounded to the storage type, as in
`workloads.py` (sigma 0.5; 1 for the fp32 shape).  A replay's buffers, descriptors and workspace are what a
training program keeps between steps, so `prepare` makes them.
"""
import math

import torch

import paper_2406_18485_amd as P
from paper_2406_18485_amd.ring import RingReplay, RingShape

DEV = "cuda:0"
CODE = {"bf16": P.BF16, "fp16": P.FP16, "fp32": P.FP32}
TORCH = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}
SIZE = {"bf16": 2, "fp16": 2, "fp32": 4}


def ring(name, part, dtype, cp, w, rank, hq, hkv, d, c, batch=1, fused=True, sigma=0.5):
    case = dict(kind="ring", part=part, dtype=dtype, cp=cp, w=w, rank=rank, hq=hq, hkv=hkv, d=d, c=c, batch=batch,
                fused=fused, sigma=sigma)
    return dict(case, name=name) if name else case


def listed():
    return [
        # the tiny fp32 shape of workloads.py: what a correctness run or a first try of the framework does;
        # every call is so short that launches and host work count
        ring("tiny_fp32_train", "train", "fp32", cp=4, w=4, rank=0, hq=2, hkv=2, d=64, c=128, sigma=1.0),
        # a short GQA sequence on a double ring, chunk no multiple of any tile: the smallest 16-bit steps
        ring("short_gqa_train", "train", "bf16", cp=4, w=2, rank=2, hq=4, hkv=1, d=128, c=200),
        # the 7B MHA shard at 32K tokens: inference-like prefill (forward alone), first rank
        ring("mha7b_32k_forward", "forward", "bf16", cp=8, w=8, rank=0, hq=8, hkv=8, d=128, c=2048),
        # the same shard, backward alone, on a rank that meets all three classes of step
        ring("mha7b_32k_backward", "backward", "bf16", cp=8, w=8, rank=4, hq=8, hkv=8, d=128, c=2048),
        # the 7B GQA shard at 128K tokens, one attention of a training step on a middle rank
        ring("gqa7b_128k_train", "train", "bf16", cp=8, w=8, rank=4, hq=4, hkv=1, d=128, c=8192),
        # the 256K double ring (4 x 4), forward replay in inner-then-outer order
        ring("dring_256k_forward", "forward", "bf16", cp=16, w=4, rank=0, hq=8, hkv=8, d=128, c=8192),
        # the 1M-token shard, forward and backward from the stored O and LSE: the largest
        ring("long_1m_train", "train", "bf16", cp=32, w=32, rank=0, hq=4, hkv=1, d=128, c=16384),
        # head_dim 64 in IEEE half (the paper's 16-bit type), odd chunk length, GQA 4:1
        ring("half_d64_train", "train", "fp16", cp=4, w=2, rank=1, hq=8, hkv=2, d=64, c=1999),
        # Attention and Update as separate calls, groups of three q heads, ragged chunks, batch of two
        ring("unfused_group3_forward", "forward", "bf16", cp=3, w=3, rank=1, hq=6, hkv=2, d=128, c=777, batch=2,
             fused=False),
        # attention without a mask, more keys than rows, forward and backward
        dict(name="full_attention_step", kind="step", dtype="bf16", batch=2, hq=8, hkv=8, d=64, q_len=1500, kv_len=4100,
             sigma=0.5),
        # Update alone on the rows of the 1M-token shard
        dict(name="update_128k_rows", kind="update", rows=131072, d=128),
        # 32 heads x 4096 tokens into and out of the messages of 4-way head parallelism, 8 KV heads replicated twice
        dict(name="head_parallel_layout", kind="layout", dtype="bf16", tokens=4096, heads=32, kv_heads=8, hp=4, rep=2, d=128),
    ]


# ------------------------------------------------------------------------------------------------ draws
MOST_FLOPS = 125e12      # the 1M-token shard
MOST_BYTES = 4e9


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    kind = rng.choices(["ring", "fp32", "step", "update", "layout"], [10, 2, 3, 1, 1])[0]
    if kind in ("ring", "fp32"):
        half = kind == "ring"
        hkv = rng.choice([1, 1, 2, 4, 8]) if half else rng.choice([1, 2])
        hq = hkv * rng.choice([1, 2, 3, 4, 8]) if half else hkv * rng.choice([1, 2, 4])
        cp = rng.choice([1, 2, 3, 4, 6, 8, 16, 32]) if half else rng.choice([1, 2, 4])
        return ring(None, rng.choice(["train", "train", "forward", "backward"]),
                    (rng.choice(["bf16", "bf16", "bf16", "fp16"]) if half else "fp32"), cp=cp,
                    w=rng.choice([x for x in range(1, cp + 1) if cp % x == 0]), rank=rng.randrange(cp), hq=hq, hkv=hkv,
                    d=(rng.choice([64, 128, 128]) if half else rng.choice([32, 64, 100, 128])),
                    c=_log(rng, 48, 16384) if half else _log(rng, 24, 512), batch=rng.choice([1, 1, 2]),
                    fused=rng.random() < 0.85, sigma=0.5 if half else 1.0)
    if kind == "step":
        hkv = rng.choice([1, 2, 8])
        return dict(kind="step", dtype=rng.choice(["bf16", "bf16", "fp16"]), batch=rng.choice([1, 2]),
                    hq=hkv * rng.choice([1, 2, 4]), hkv=hkv, d=rng.choice([64, 128]), q_len=_log(rng, 32, 16384),
                    kv_len=_log(rng, 64, 32768), sigma=0.5)
    if kind == "update":
        return dict(kind="update", rows=_log(rng, 512, 400000), d=rng.choice([64, 128]))
    hp = rng.choice([2, 4, 8])
    return dict(kind="layout", dtype=rng.choice(["bf16", "fp16"]), tokens=_log(rng, 500, 16384), heads=32, kv_heads=8,
                hp=hp, rep=rng.choice([2, 4]), d=rng.choice([64, 128]))


def draw(rng):
    while True:
        case = _draw_once(rng)
        w = work(case)
        if w["flops"] <= MOST_FLOPS and w["bytes"] <= MOST_BYTES:
            return case


# --------------------------------------------------------------------------------------------- the work
def _pairs(case):
    """Visible (query, key) pairs per q head and batch element: a rank of the ring sees half of every other
    rank's block and the causal half of its own."""
    if case["kind"] == "step":
        return case["q_len"] * case["kv_len"]
    L = 2 * case["c"]
    return L * (L + 1) // 2 + (case["cp"] - 1) * (L * L // 2)


def work(case):
    kind = case["kind"]
    if kind == "update":
        return {"bytes": case["rows"] * (12 * case["d"] + 12), "flops": 3 * case["rows"] * case["d"]}
    e = SIZE[case["dtype"]]
    if kind == "layout":
        q = case["tokens"] * case["heads"] * case["d"]            # packed, then unpacked
        kv = case["tokens"] * case["kv_heads"] * case["d"]        # K and V: read once, written `rep` times
        grad = (case["rep"] + 1) * 4 * kv                         # the replicas' fp32 gradients, read; the sum, written
        return {"bytes": 4 * q * e + 2 * kv * e * (1 + case["rep"]) + 2 * grad, "flops": 2 * (case["rep"] - 1) * kv}
    ring_ = kind == "ring"
    part = case["part"] if ring_ else "train"
    lq = 2 * case["c"] if ring_ else case["q_len"]
    lk = 2 * case["c"] * case["cp"] if ring_ else case["kv_len"]
    rows, d = case["batch"] * case["hq"] * lq, case["d"]
    keys = case["batch"] * case["hkv"] * lk
    pairs = case["batch"] * case["hq"] * _pairs(case)
    nbytes = flops = 0
    if part != "backward":   # q, k, v in; fp32 out, lse and the stored o
        nbytes += rows * d * e + 2 * keys * d * e + rows * (4 * d + 4 + d * e)
        flops += 4 * d * pairs
    if part != "forward":    # q, o, d_o, k, v, lse in; dq, dk, dv
        nbytes += 3 * rows * d * e + 4 * rows + 2 * keys * d * e + 4 * d * (rows + 2 * keys)
        flops += 10 * d * pairs
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the distance from the same attention in 64 bits, measured over the listed and drawn
    shapes (the long ones with shorter chunks): 2.7e-3 for bf16, 3.1e-4 for half, where probabilities, score
    gradients and the stored O are rounded to the 16-bit type, 8.8e-7 for fp32, where only the sums differ;
    largest single differences 0.19, 7e-3 and 1.2e-5 of the result's root mean square (gradients of the first
    keys of a causal sequence, which grow with its length)."""
    if case["kind"] == "layout":    # copies, and sums whose order is part of the contract
        return "exact"
    if case["kind"] == "update":    # 5e-8 and 3.3e-7 measured for one merge; passes merge again into the same rows
        return {"rel": 4e-7, "max": 3e-6}
    return {"fp32": {"rel": 4e-6, "max": 5e-5}, "fp16": {"rel": 1.3e-3, "max": 0.1}, "bf16": {"rel": 1.1e-2, "max": 0.8}}[case["dtype"]]


# ------------------------------------------------------------------------------------------------- runs
def _normal(gen, shape, sigma, dtype):
    return (torch.randn(shape, device=DEV, generator=gen) * sigma).to(TORCH[dtype])


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    return {"ring": _prepare_ring, "step": _prepare_step, "update": _prepare_update, "layout": _prepare_layout}[case["kind"]](case, gen)


def run(state):
    return state["run"](state)


def _prepare_ring(case, gen):
    B, L, d = case["batch"], 2 * case["c"], case["d"]
    q = _normal(gen, (B, case["hq"], L, d), case["sigma"], case["dtype"])
    d_o = _normal(gen, (B, case["hq"], L, d), case["sigma"], case["dtype"])
    k = torch.empty(case["cp"], B, case["hkv"], L, d, dtype=TORCH[case["dtype"]], device=DEV)
    v = torch.empty_like(k)
    for s in range(case["cp"]):   # one source rank at a time: the fp32 draws stay small
        k[s] = _normal(gen, k.shape[1:], case["sigma"], case["dtype"])
        v[s] = _normal(gen, k.shape[1:], case["sigma"], case["dtype"])
    rep = RingReplay(RingShape(cp=case["cp"], w=case["w"], rank=case["rank"], hq=case["hq"], hkv=case["hkv"], d=d,
                               c=case["c"], dtype=CODE[case["dtype"]], scale=1.0 / math.sqrt(d), batch=B), DEV)
    if case["part"] == "backward":   # the stored O and LSE of the forward pass
        rep.forward(q, k, v)
    return {"run": _run_ring, "part": case["part"], "fused": case["fused"], "rep": rep, "q": q, "k": k, "v": v, "d_o": d_o}


def _run_ring(s):
    rep, out = s["rep"], {}
    if s["part"] != "backward":
        rep.forward(s["q"], s["k"], s["v"], fuse_merge=s["fused"])
        out.update(out=rep.out, lse=rep.lse, o=rep.o)
    if s["part"] != "forward":
        rep.backward(s["q"], s["k"], s["v"], s["d_o"])
        out.update(dq=rep.dq, dk=rep.dk, dv=rep.dv)
    return out


def _prepare_step(case, gen):
    B, d, lq, lk = case["batch"], case["d"], case["q_len"], case["kv_len"]
    q_shape, k_shape = (B, case["hq"], lq, d), (B, case["hkv"], lk, d)
    s = {"run": _run_step, "dtype": CODE[case["dtype"]], "rows": B * case["hq"] * lq, "d": d}
    for name, shape in (("q", q_shape), ("k", k_shape), ("v", k_shape), ("d_o", q_shape)):
        s[name] = _normal(gen, shape, case["sigma"], case["dtype"])
    f32 = dict(dtype=torch.float32, device=DEV)
    s["out"], s["dq"] = torch.empty(q_shape, **f32), torch.empty(q_shape, **f32)
    s["dk"], s["dv"] = torch.empty(k_shape, **f32), torch.empty(k_shape, **f32)
    s["lse"], s["delta"] = torch.empty(q_shape[:3], **f32), torch.empty(q_shape[:3], **f32)
    s["o"] = torch.empty(q_shape, dtype=TORCH[case["dtype"]], device=DEV)
    desc = dict(batch=B, n_q_heads=case["hq"], n_kv_heads=case["hkv"], head_dim=d, q_len=lq, kv_len=lk,
                dtype=s["dtype"], softmax_scale=1.0 / math.sqrt(d))
    s["fwd"], s["bwd"] = P.make_desc(**desc), P.make_desc(**desc, flags=P.COMPUTE_DELTA)
    s["workspace"] = torch.empty(max(P.workspace_bytes(s["bwd"]), 16), dtype=torch.uint8, device=DEV)
    return s


def _run_step(s):
    P.attn_step_fwd(s["fwd"], s["q"], s["k"], s["v"], s["out"], s["lse"])
    P.finalize_out(s["rows"], s["d"], s["out"], s["o"], s["dtype"])
    s["dq"].zero_()
    P.attn_step_bwd(s["bwd"], s["q"], s["k"], s["v"], s["o"], s["d_o"], s["lse"], s["delta"], s["dq"], s["dk"], s["dv"],
                    s["workspace"])
    return {n: s[n] for n in ("out", "lse", "o", "dq", "dk", "dv")}


def _prepare_update(case, gen):
    rows, d = case["rows"], case["d"]
    s = {"run": _run_update, "rows": rows, "d": d}
    for side in ("", "block_"):
        s[side + "out"] = torch.randn(rows, d, device=DEV, generator=gen) * 0.1
        s[side + "lse"] = 8.0 + torch.randn(rows, device=DEV, generator=gen) * 0.2
    return s


def _run_update(s):
    P.lse_merge(s["rows"], s["d"], s["out"], s["lse"], s["block_out"], s["block_lse"])
    return {"out": s["out"], "lse": s["lse"]}


def _prepare_layout(case, gen):
    t, h, d, hp, rep, kvh = (case[n] for n in ("tokens", "heads", "d", "hp", "rep", "kv_heads"))
    e, hl = SIZE[case["dtype"]], case["heads"] // case["hp"]
    half = dict(dtype=TORCH[case["dtype"]], device=DEV)
    s = {"run": _run_layout, "row_bytes": d * e, "kv_heads": kvh, "rep": rep, "per_head": t * d,
         "x": _normal(gen, (t, h, d), 0.5, case["dtype"]), "messages": torch.empty(hp, hl, t, d, **half),
         "received": _normal(gen, (hp, hl, t, d), 0.5, case["dtype"]), "local": torch.empty(hl, hp * t, d, **half),
         "kv": [_normal(gen, (kvh, t, d), 0.5, case["dtype"]) for _ in range(2)],
         "kv_rep": [torch.empty(kvh * rep, t, d, **half) for _ in range(2)],
         "g_rep": [torch.randn(kvh * rep, t, d, device=DEV, generator=gen) for _ in range(2)],
         "g": [torch.empty(kvh, t, d, device=DEV) for _ in range(2)]}
    s["pack"] = ((hp, hl, t), (hl * d * e, d * e, h * d * e), (hl * t * d * e, t * d * e, d * e))
    s["unpack"] = ((hp, hl, t), (hl * t * d * e, t * d * e, d * e), (t * d * e, hp * t * d * e, d * e))
    s["replicate"] = ((kvh, rep, t), (t * d * e, 0, d * e), (rep * t * d * e, t * d * e, d * e))
    return s


def _run_layout(s):
    P.permute_rows(*s["pack"], s["row_bytes"], s["x"], s["messages"])
    P.permute_rows(*s["unpack"], s["row_bytes"], s["received"], s["local"])
    for i in range(2):   # K and V
        P.permute_rows(*s["replicate"], s["row_bytes"], s["kv"][i], s["kv_rep"][i])
        P.reduce_replicas(s["kv_heads"], s["rep"], s["per_head"], s["g_rep"][i], s["g"][i])
    return {"messages": s["messages"], "local": s["local"], "kv": s["kv_rep"], "grad": s["g"]}
