"""The calls whose speed counts: passes of pipeline stages and single operations.

Each case is what a training program does with this library on one GPU,
through its public entry points, at sizes of the workloads in synth/ and of
the tests, or at generic ones:

  stage       one optimizer step's gradient work of a stage: the gradient
              bucket zeroed, then an Order of forward and backward passes over
              its microbatches (the weights, the workspace and the microbatch
              buffers are what such a program keeps)
  attention   causal attention, forward then backward
  mlp         the six products of a SwiGLU block, forward then backward
  rmsnorm     RMSNorm, forward then backward
  adam        the AdamW step over a flat shard, with the bf16 cast
  accumulate  a microbatch's gradient added into the fp32 bucket
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

from paper_2606_11169_amd import libchunk as lc
from paper_2606_11169_amd.runner import random_stage

DEV = "cuda"
DTYPES = {"fp32": (torch.float32, lc.LC_FP32), "bf16": (torch.bfloat16, lc.LC_BF16),
          "fp16": (torch.float16, lc.LC_FP16)}


def _stage(name, dtype, layers, heads, hd, ffn, seq, batch, mbs, kv=0, qk_norm=False, experts=0,
           order="1f1b"):
    return {"name": name, "kind": "stage", "dtype": dtype, "layers": layers, "heads": heads,
            "hd": hd, "kv": kv, "qk_norm": qk_norm, "ffn": ffn, "experts": experts, "seq": seq,
            "batch": batch, "mbs": mbs, "order": order}


def listed():
    return [
        # the tiny fp32 stage's whole step: small launches back to back, as a
        # user meets it when checking a setup in full precision
        _stage("tiny_fp32_step", "fp32", 2, 4, 32, 344, 64, 2, 4),
        # a small model trained in fp32, ragged sequence length
        _stage("fp32_layer_d768", "fp32", 1, 12, 64, 2048, 200, 2, 2),
        # a small bf16 stage: few tiles per product, many launches per step
        _stage("small_bf16_step", "bf16", 2, 4, 128, 1408, 256, 1, 4),
        # a layer of the Llama-style d-2048 stage, two microbatches accumulated
        _stage("llama2k_layer", "bf16", 1, 16, 128, 5632, 2048, 1, 2),
        # a layer of the 7B-shaped stage (the benchmark's), forward and backward
        _stage("stage7b_layer", "bf16", 1, 32, 128, 11008, 4096, 1, 1),
        # a layer of the Qwen3-8B-shaped stage (grouped-query attention, q/k
        # norm) with the backward split into its input and weight passes
        _stage("qwen3_split_layer", "bf16", 1, 32, 128, 12288, 4096, 1, 1, kv=8, qk_norm=True,
               order="split"),
        # a layer of the mixture-of-experts stage, weight passes overlapped
        # with the next input pass on a second stream (the benchmark's Order)
        _stage("moe_overlap_layer", "bf16", 1, 16, 128, 1408, 2048, 2, 3, experts=8,
               order="overlap"),
        # grouped-query attention called by itself, two sequences of 15 blocks
        {"name": "attention_gqa_s1920", "kind": "attention", "dtype": "fp16", "batch": 2,
         "seq": 1920, "heads": 16, "kv": 4},
        # a SwiGLU block over a ragged number of tokens (a packed microbatch)
        {"name": "mlp_t1003", "kind": "mlp", "tokens": 1003, "d": 2048, "ffn": 5632},
        # rows of a 40-head model, ragged number of tokens
        {"name": "rmsnorm_t3001_d5120", "kind": "rmsnorm", "tokens": 3001, "d": 5120},
        # an eighth of the 1.6e9-element AdamW shard, odd length
        {"name": "adam_2e8", "kind": "adam", "n": 200_000_001},
        # a data-parallel rank's share of the 7B-shaped bucket, bf16 gradients
        {"name": "accumulate_1e8", "kind": "accumulate", "dtype": "bf16", "n": 101_190_003},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _mult(x, m, lo):
    return max(lo, m * round(x / m))


def _divisor(rng, n):
    return rng.choice([k for k in range(1, n + 1) if n % k == 0])


def draw(rng):
    kind = rng.choice(["stage"] * 6 + ["attention", "attention", "mlp", "mlp", "rmsnorm", "adam",
                                       "accumulate"])
    while True:
        if kind == "stage":
            variant = rng.choice(["fp32", "dense", "dense", "gqa", "moe"])
            order = rng.choice(["1f1b", "1f1b", "split", "overlap", "zero2"])
            mbs = rng.randint(2 if order == "overlap" else 1, 4)
            layers = rng.randint(1, 2)
            if variant == "fp32":
                heads, hd = rng.randint(2, 12), rng.choice([16, 32, 64])
                kv = _divisor(rng, heads) if rng.random() < 0.3 else 0
                c = _stage("", "fp32", layers, heads, hd,
                           int(heads * hd * rng.uniform(2, 4)), int(_log(rng, 24, 320)),
                           rng.randint(1, 2), mbs, kv=kv, qk_norm=kv > 0, order=order)
            else:
                heads = round(_log(rng, 2, 32))
                d = 128 * heads
                moe = variant == "moe"
                ffn = _mult(d * (rng.uniform(0.5, 1.5) if moe else rng.uniform(2.2, 3.5)), 64, 64)
                kv = _divisor(rng, heads) if variant == "gqa" else 0
                c = _stage("", "bf16", layers, heads, 128, ffn,
                           _mult(_log(rng, 128, 4096), 128, 128), rng.randint(1, 2), mbs, kv=kv,
                           qk_norm=kv > 0, experts=rng.choice([2, 4, 8, 16]) if moe else 0,
                           order=order)
            fits = work(c)["flops"] <= (6e10 if variant == "fp32" else 2e12) and \
                work(c)["bytes"] <= 6e9
        elif kind == "attention":
            heads = round(_log(rng, 2, 32))
            c = {"kind": kind, "dtype": rng.choice(["fp16", "bf16"]), "batch": rng.randint(1, 4),
                 "seq": _mult(_log(rng, 128, 8192), 128, 128), "heads": heads,
                 "kv": _divisor(rng, heads) if rng.random() < 0.5 else heads}
            fits = work(c)["flops"] <= 1e12
        elif kind == "mlp":
            d = _mult(_log(rng, 256, 4096), 8, 256)
            c = {"kind": kind, "tokens": round(_log(rng, 8, 8192)), "d": d,
                 "ffn": _mult(d * rng.uniform(2.2, 3.5), 64, 64)}
            fits = work(c)["flops"] <= 2e12
        elif kind == "rmsnorm":
            c = {"kind": kind, "tokens": round(_log(rng, 1, 16384)),
                 "d": _mult(_log(rng, 256, 8192), 8, 256)}
            fits = c["tokens"] * c["d"] <= 1 << 26
        else:
            c = {"kind": kind, "n": round(_log(rng, 1000, 4e8))}
            if kind == "accumulate":
                c["dtype"] = rng.choice(["bf16", "fp32"])
            fits = True
        c.pop("name", None)
        if fits:
            return c


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _randn(g, shape, std, dtype):
    return torch.randn(shape, generator=g, device=DEV).mul_(std).to(dtype)


def _desc(c):
    moe = c["experts"] > 0
    return lc.make_desc(c["layers"], c["heads"] * c["hd"], c["heads"], c["hd"],
                        0 if moe else c["ffn"], c["seq"], c["batch"], c["dtype"] == "bf16",
                        n_experts=c["experts"], top_k=2 if moe else 0,
                        d_ff_expert=c["ffn"] if moe else 0, n_kv_heads=c["kv"],
                        qk_norm=c["qk_norm"])


def _layout(c):
    """(name, shape) of a layer's tensors in the flat bucket, in its order."""
    d, f, hd = c["heads"] * c["hd"], c["ffn"], c["hd"]
    dkv = (c["kv"] or c["heads"]) * hd
    out = [("wq", (d, d)), ("wk", (dkv, d)), ("wv", (dkv, d)), ("wo", (d, d)), ("g1", (d,))]
    if c["qk_norm"]:
        out += [("qn", (hd,)), ("kn", (hd,))]
    if c["experts"]:
        out.append(("wr", (c["experts"], d)))
        for e in range(c["experts"]):
            out += [(f"w1_{e}", (f, d)), (f"w3_{e}", (f, d)), (f"w2_{e}", (d, f))]
    else:
        out += [("w1", (f, d)), ("w3", (f, d)), ("w2", (d, f))]
    return out + [("g2", (d,))]


def _stage_inputs(c, seed):
    """Flat weights (matrices N(0, 0.02), gains about 1) and N(0, 1) X, dY. The
    tokens of a mixture of experts lean towards two experts in every layer, some
    experts wanted more than others, as a trained router's do: the two largest
    logits then stand clear of the rest, and rounding does not change the
    routing."""
    dt = DTYPES[c["dtype"]][0]
    g = _gen(seed)
    n = sum(math.prod(s) for _, s in _layout(c))
    w = _randn(g, c["layers"] * n, 0.02, dt)
    off, routers = 0, []
    for _ in range(c["layers"]):
        for name, shape in _layout(c):
            k = math.prod(shape)
            if len(shape) == 1:
                w[off:off + k] = _randn(g, k, 0.1, torch.float32).add_(1.0).to(dt)
            if name == "wr":
                routers.append(F.normalize(w[off:off + k].view(shape).float()))
            off += k
    shape = (c["batch"], c["seq"], c["heads"] * c["hd"])
    xs = []
    for _ in range(c["mbs"]):
        x = _randn(g, shape, 1.0, torch.float32)
        for u in routers:
            share = torch.arange(1, len(u) + 1, dtype=torch.float32, device=DEV) / len(u) + 1
            pick = torch.multinomial(share.expand(shape[0] * shape[1], -1), 2, generator=g)
            x += (8 * u[pick[:, 0]] + 6 * u[pick[:, 1]]).view(shape)
        xs.append(x.to(dt))
    dys = [_randn(g, shape, 1.0, dt) for _ in range(c["mbs"])]
    return w, xs, dys


def _entries(c):
    M, P = c["mbs"], 2
    if c["order"] == "split":
        return lc.lc_order_1f1b_split(M, P, 0, 0)
    if c["order"] == "overlap":
        return lc.lc_order_1f1b_split_overlap(M, P, 0, 1)
    return lc.lc_order_1f1b(M, P, 0)


def _shard(c, n):
    """A quarter of the bucket (the last one but one), as rank 2 of 4 holds it."""
    k = n // 4 // 4 * 4
    return 2 * k, k


def _qkv_cols(c):
    return (c["heads"] + 2 * c["kv"]) * 128


def _rope(seq, half, base=10000.0):
    ang = torch.arange(seq, dtype=torch.float64, device=DEV)[:, None] * base ** (
        -torch.arange(half, dtype=torch.float64, device=DEV) / half)
    return torch.cos(ang), torch.sin(ang)


def _attention_inputs(c, seed):
    g = _gen(seed)
    T = c["batch"] * c["seq"]
    qkv = _randn(g, (T, _qkv_cols(c)), 1.0, DTYPES[c["dtype"]][0])
    return qkv, _randn(g, (T, c["heads"] * 128), 1.0, torch.bfloat16)


def _mlp_inputs(c, seed):
    g = _gen(seed)
    T, d, f = c["tokens"], c["d"], c["ffn"]
    return {"x": _randn(g, (T, d), 1.0, torch.bfloat16), "h": _randn(g, (T, d), 1.0, torch.float32),
            "w13": _randn(g, (2 * f, d), 0.02, torch.bfloat16),
            "w2": _randn(g, (d, f), 0.02, torch.bfloat16),
            "dy": _randn(g, (T, d), 1.0, torch.bfloat16)}


def _norm_inputs(c, seed):
    g = _gen(seed)
    T, d = c["tokens"], c["d"]
    return {"x": _randn(g, (T, d), 1.0, torch.float32),
            "g": _randn(g, (d,), 0.1, torch.float32).add_(1.0).to(torch.bfloat16),
            "dn": _randn(g, (T, d), 1.0, torch.float32),
            "dres": _randn(g, (T, d), 1.0, torch.float32)}


def _adam_inputs(c, seed):
    g = _gen(seed)
    n = c["n"]
    return {"p": _randn(g, n, 0.02, torch.float32), "m": _randn(g, n, 1e-3, torch.float32),
            "v": _randn(g, n, 1e-3, torch.float32).square_(),
            "g": _randn(g, n, 1e-3, torch.bfloat16)}


ADAM_HP = (3e-4, 0.9, 0.95, 1e-8, 0.1, 10)  # lr, beta1, beta2, eps, weight decay, step


def _acc_inputs(c, seed):
    g = _gen(seed)
    return {"a": _randn(g, c["n"], 1.0, torch.float32),
            "g": _randn(g, c["n"], 1.0, DTYPES[c["dtype"]][0])}


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "stage":
        w, xs, dys = _stage_inputs(c, seed)
        entries = _entries(c)
        _, peak, peak_w = lc.lc_order_validate_split(entries, c["mbs"], c["mbs"], c["mbs"])
        r = random_stage(_desc(c), peak, max_w_pending=peak_w)
        r.m = r.v = r.master = None  # no optimizer step here
        r.w = w
        r.X, r.dY = xs, dys
        r.Y, r.dX = [torch.empty_like(x) for x in xs], [torch.empty_like(x) for x in xs]
        s = {"r": r, "entries": entries}
        if c["order"] == "overlap":
            s["aux"] = torch.cuda.Stream()
        if c["order"] == "zero2":
            s["off"], k = _shard(c, r.n_params)
            s["shard"] = torch.zeros(k, dtype=torch.float32, device=DEV)
    elif kind == "attention":
        qkv, dout = _attention_inputs(c, seed)
        B, S, H, kv = c["batch"], c["seq"], c["heads"], c["kv"]
        cos, sin = (t.float() for t in _rope(S, 64))
        nb = lc.lc_attention_scratch_bytes(B, S, H, kv)
        s = {"qkv": qkv, "dout": dout, "cos": cos, "sin": sin, "scratch_bytes": nb,
             "scratch": torch.empty(nb, dtype=torch.uint8, device=DEV),
             "o": torch.empty_like(dout), "dqkv": torch.empty_like(qkv, dtype=torch.bfloat16),
             "lse": torch.empty((B, H, S), dtype=torch.float32, device=DEV)}
    elif kind == "mlp":
        s = _mlp_inputs(c, seed)
        T, d, f = c["tokens"], c["d"], c["ffn"]
        for k, shape, dt in (("gate", (T, f), torch.float32), ("up", (T, f), torch.float32),
                             ("act", (T, f), torch.bfloat16), ("y", (T, d), torch.float32),
                             ("da", (T, 2 * f), torch.bfloat16), ("dx", (T, d), torch.float32),
                             ("grad", (3 * f * d,), torch.float32)):
            s[k] = torch.empty(shape, dtype=dt, device=DEV)
    elif kind == "rmsnorm":
        s = _norm_inputs(c, seed)
        T, d = c["tokens"], c["d"]
        s["n"] = torch.empty((T, d), dtype=torch.bfloat16, device=DEV)
        s["rstd"] = torch.empty(T, dtype=torch.float32, device=DEV)
        s["dx"] = torch.empty((T, d), dtype=torch.float32, device=DEV)
        s["dx16"] = torch.empty((T, d), dtype=torch.bfloat16, device=DEV)
        s["dg"] = torch.zeros(d, dtype=torch.float32, device=DEV)
        s["scratch_bytes"] = lc.lc_rmsnorm_scratch_bytes(T, d)
        s["scratch"] = torch.empty(s["scratch_bytes"], dtype=torch.uint8, device=DEV)
    elif kind == "adam":
        s = _adam_inputs(c, seed)
        s["out"] = torch.empty(c["n"], dtype=torch.bfloat16, device=DEV)
    else:
        s = _acc_inputs(c, seed)
    s["case"] = c
    return s


# ------------------------------------------------------------------ the pass

def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "stage":
        r = s["r"]
        if c["order"] == "zero2":
            lc.lc_zero_fill_f32(s["shard"], s["shard"].numel(), r.stream)
            r.run_order_zero(s["entries"], 2, s["shard"], s["off"], r.grad)
            return {"y": r.Y, "dx": r.dX, "grad": s["shard"]}
        r.zero_grad()
        r.run_order(s["entries"], s.get("aux"))
        return {"y": r.Y, "dx": r.dX, "grad": r.grad}
    if kind == "attention":
        B, S, H, kv, ld = c["batch"], c["seq"], c["heads"], c["kv"], _qkv_cols(c)
        dt, es = DTYPES[c["dtype"]][1], 2
        q = s["qkv"].data_ptr()
        k, v = q + H * 128 * es, q + (H + kv) * 128 * es
        dq = s["dqkv"].data_ptr()
        dk, dv = dq + H * 128 * 2, dq + (H + kv) * 128 * 2
        lc.lc_attention_forward(dt, lc.LC_BF16, B, S, H, 128, q, k, v, ld, s["o"], H * 128,
                                s["lse"], Hkv=kv)
        lc.lc_attention_backward(dt, lc.LC_BF16, B, S, H, 128, q, k, v, ld, s["o"], s["dout"],
                                 H * 128, s["lse"], dq, dk, dv, ld, s["cos"], s["sin"],
                                 s["scratch"], s["scratch_bytes"], Hkv=kv)
        return {"o": s["o"], "lse": s["lse"], "dqkv": s["dqkv"]}
    if kind == "mlp":
        T, d, f = c["tokens"], c["d"], c["ffn"]
        bf, f32 = lc.LC_BF16, lc.LC_FP32
        g13, g2 = s["grad"].data_ptr(), s["grad"].data_ptr() + 2 * f * d * 4
        lc.lc_zero_fill_f32(s["grad"], 3 * f * d)
        # forward: gate/up with SwiGLU, then down with the residual
        lc.lc_gemm(bf, lc.LC_EPI_SWIGLU, T, f, d, s["x"], d, 1, s["w13"], d, 1, s["act"], f,
                   aux0=s["gate"], aux1=s["up"], ld_aux=f, aux_dtype=f32)
        lc.lc_gemm(bf, lc.LC_EPI_RESIDUAL, T, d, f, s["act"], f, 1, s["w2"], f, 1, s["y"], d,
                   R=s["h"], ldr=d, c_dtype=f32, r_dtype=f32)
        # backward: dgate|dup, dW2, dx, dW1|dW3
        lc.lc_gemm(bf, lc.LC_EPI_SWIGLU_BWD, T, f, d, s["dy"], d, 1, s["w2"], f, 0, s["da"], 2 * f,
                   aux0=s["gate"], aux1=s["up"], ld_aux=f, aux_dtype=f32)
        lc.lc_gemm(bf, lc.LC_EPI_ACCUM_F32, d, f, T, s["dy"], d, 0, s["act"], f, 0, g2, f)
        lc.lc_gemm(bf, lc.LC_EPI_STORE, T, d, 2 * f, s["da"], 2 * f, 1, s["w13"], d, 0, s["dx"], d,
                   c_dtype=f32)
        lc.lc_gemm(bf, lc.LC_EPI_ACCUM_F32, 2 * f, d, T, s["da"], 2 * f, 0, s["x"], d, 0, g13, d)
        return {"y": s["y"], "act": s["act"], "da": s["da"], "dx": s["dx"], "grad": s["grad"]}
    if kind == "rmsnorm":
        T, d = c["tokens"], c["d"]
        bf, f32 = lc.LC_BF16, lc.LC_FP32
        lc.lc_zero_fill_f32(s["dg"], d)
        lc.lc_rmsnorm_forward(T, d, s["x"], s["g"], 1e-5, s["n"], s["rstd"], f32, bf, bf)
        lc.lc_rmsnorm_backward(T, d, s["dn"], s["x"], s["rstd"], s["g"], s["dres"], s["dx"],
                               s["dg"], s["scratch"], s["scratch_bytes"], f32, f32, bf, f32, f32,
                               dx_copy=s["dx16"])
        return {k: s[k] for k in ("n", "rstd", "dx", "dx16", "dg")}
    if kind == "adam":
        lc.shard_adam_step(s["p"], s["m"], s["v"], s["g"], lc.LC_BF16, s["out"], c["n"], *ADAM_HP)
        return {k: s[k] for k in ("p", "m", "v", "out")}
    lc.chunk_accumulate_grad(s["a"], s["g"], DTYPES[c["dtype"]][1], c["n"])
    return s["a"]


# ------------------------------------------------------------------ work

def work(case):
    c, kind = case, case["kind"]
    if kind == "stage":
        es = 2 if c["dtype"] == "bf16" else 4
        d = c["heads"] * c["hd"]
        dkv = (c["kv"] or c["heads"]) * c["hd"]
        T = c["batch"] * c["seq"]
        n = c["layers"] * sum(math.prod(s) for _, s in _layout(c))
        ffn = 6 * c["ffn"] * d * (2 if c["experts"] else 1) + 2 * c["experts"] * d
        fwd = T * (2 * d * (2 * d + 2 * dkv) + ffn) + \
            2 * c["batch"] * c["heads"] * c["hd"] * c["seq"] * (c["seq"] + 1)
        return {"flops": 3.0 * fwd * c["layers"] * c["mbs"],
                "bytes": float(n * (es + 4) + 4 * c["mbs"] * T * d * es)}
    if kind == "attention":
        pairs = c["batch"] * c["heads"] * c["seq"] * (c["seq"] + 1) / 2
        T = c["batch"] * c["seq"]
        return {"flops": 3 * 4 * 128 * pairs,
                "bytes": T * (2.0 * 2 * _qkv_cols(c) + 2 * 2 * c["heads"] * 128 + 4 * c["heads"])}
    if kind == "mlp":
        T, d, f = c["tokens"], c["d"], c["ffn"]
        return {"flops": 18.0 * T * d * f,
                "bytes": T * (d * (2.0 + 4 + 2 + 4 + 4) + f * (2 + 4)) + 3 * d * f * (2 + 4)}
    if kind == "rmsnorm":
        T, d = c["tokens"], c["d"]
        return {"flops": 15.0 * T * d, "bytes": T * d * (4.0 * 3 + 4 + 2 + 2) + 4 * T + 6 * d}
    if kind == "adam":
        return {"flops": 16.0 * c["n"], "bytes": 28.0 * c["n"]}
    return {"flops": 1.0 * c["n"], "bytes": (10.0 if c["dtype"] == "bf16" else 12.0) * c["n"]}


def tolerance(case):
    c, kind = case, case["kind"]
    if kind in ("adam", "accumulate"):
        return "exact"  # defined operation by operation
    # four times the error against 64 bits, which is at most 8e-7 (fp32 stages),
    # 4e-3 (bf16 stages), 3e-3 (attention) and 1.7e-3 (mlp, rmsnorm: the bf16
    # rounding of the outputs)
    if kind == "stage":
        return {"rel": 5e-6} if c["dtype"] == "fp32" else {"rel": 1.6e-2}
    return {"rel": 1.2e-2} if kind == "attention" else {"rel": 7e-3}


# ------------------------------------------------------------------ 64 bits

def _rotate(x, cos, sin):
    a, b = x.chunk(2, dim=-1)
    return torch.cat([a * cos - b * sin, a * sin + b * cos], dim=-1)


def _norm64(x, g, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * g


def _causal64(q, k, v):
    """softmax(q k^T / sqrt(hd)) v of one head, [S, hd] each."""
    S = q.shape[0]
    mask = torch.ones((S, S), dtype=torch.bool, device=q.device).triu(1)
    sc = (q @ k.t() / math.sqrt(q.shape[1])).masked_fill_(mask, -math.inf)
    return torch.softmax(sc, -1) @ v, torch.logsumexp(sc, -1)


def _layer64(c, P, x):
    d, hd, H = c["heads"] * c["hd"], c["hd"], c["heads"]
    kv, B, S, eps = c["kv"] or H, c["batch"], c["seq"], 1e-5
    cos, sin = _rope(S, hd // 2)
    n1 = _norm64(x, P["g1"], eps)
    q, k, v = ((n1 @ P[w].t()).view(B, S, -1, hd) for w in ("wq", "wk", "wv"))
    if c["qk_norm"]:
        q, k = _norm64(q, P["qn"], eps), _norm64(k, P["kn"], eps)
    q, k = (_rotate(t, cos[:, None], sin[:, None]) for t in (q, k))
    o = torch.stack([torch.stack([_causal64(q[b, :, h], k[b, :, h * kv // H], v[b, :, h * kv // H])[0]
                                  for h in range(H)], 1) for b in range(B)]).view(B * S, d)
    h = x + o @ P["wo"].t()
    n2 = _norm64(h, P["g2"], eps)
    if not c["experts"]:
        return h + (F.silu(n2 @ P["w1"].t()) * (n2 @ P["w3"].t())) @ P["w2"].t()
    probs, sel = torch.softmax(n2 @ P["wr"].t(), -1).topk(2, -1)
    probs = probs / probs.sum(-1, keepdim=True)
    y = h
    for e in range(c["experts"]):
        t, j = torch.nonzero(sel == e, as_tuple=True)
        n = n2[t]
        f = (F.silu(n @ P[f"w1_{e}"].t()) * (n @ P[f"w3_{e}"].t())) @ P[f"w2_{e}"].t()
        y = y.index_add(0, t, probs[t, j][:, None] * f)
    return y


def exact(case, seed):
    c, kind = case, case["kind"]
    f64 = torch.float64
    if kind == "stage":
        w, xs, dys = _stage_inputs(c, seed)
        n = w.numel() // c["layers"]
        flat = w.to(f64)
        layers, off = [], 0
        for _ in range(c["layers"]):
            P = {}
            for name, shape in _layout(c):
                k = math.prod(shape)
                P[name] = flat[off:off + k].view(shape).requires_grad_()
                off += k
            layers.append(P)
        ys, dxs = [], []
        for x, dy in zip(xs, dys):
            x0 = x.to(f64).view(-1, x.shape[-1]).requires_grad_()
            y = x0
            for P in layers:
                y = _layer64(c, P, y)
            y.backward(dy.to(f64).view(y.shape))
            ys.append(y.detach().view(x.shape))
            dxs.append(x0.grad.view(x.shape))
            del y
        grad = torch.cat([torch.zeros(math.prod(s), dtype=f64, device=DEV) if P[name].grad is None
                          else P[name].grad.reshape(-1) for P in layers for name, s in _layout(c)])
        if c["order"] == "zero2":
            o, k = _shard(c, c["layers"] * n)
            grad = grad[o:o + k]
        return {"y": ys, "dx": dxs, "grad": grad}
    if kind == "attention":
        qkv, dout = _attention_inputs(c, seed)
        B, S, H, kv = c["batch"], c["seq"], c["heads"], c["kv"]
        cos, sin = _rope(S, 64)
        x = qkv.to(f64).view(B, S, H + 2 * kv, 128)
        do = dout.to(f64).view(B, S, H, 128)
        o = torch.empty_like(do)
        lse = torch.empty((B, H, S), dtype=f64, device=DEV)
        dx = torch.zeros_like(x)
        for b in range(B):
            for h in range(H):
                j = H + h * kv // H
                t = [x[b, :, i].clone().requires_grad_() for i in (h, j, j + kv)]
                oh, lh = _causal64(*t)
                oh.backward(do[b, :, h])
                o[b, :, h], lse[b, h] = oh.detach(), lh.detach()
                # q and k are given rotated; their gradients come rotated back
                dx[b, :, h] = _rotate(t[0].grad, cos, -sin)
                dx[b, :, j] += _rotate(t[1].grad, cos, -sin)
                dx[b, :, j + kv] += t[2].grad
        return {"o": o.view(B * S, -1), "lse": lse, "dqkv": dx.view(B * S, -1)}
    if kind == "mlp":
        i = {k: v.to(f64) for k, v in _mlp_inputs(c, seed).items()}
        f = c["ffn"]
        g, u = i["x"] @ i["w13"][:f].t(), i["x"] @ i["w13"][f:].t()
        sg = torch.sigmoid(g)
        act = g * sg * u
        dact = i["dy"] @ i["w2"]
        da = torch.cat([dact * u * sg * (1 + g * (1 - sg)), dact * g * sg], -1)
        return {"y": i["h"] + act @ i["w2"].t(), "act": act, "da": da, "dx": da @ i["w13"],
                "grad": torch.cat([(da.t() @ i["x"]).reshape(-1), (i["dy"].t() @ act).reshape(-1)])}
    if kind == "rmsnorm":
        i = {k: v.to(f64) for k, v in _norm_inputs(c, seed).items()}
        r = torch.rsqrt(i["x"].square().mean(-1, keepdim=True) + 1e-5)
        xh, dxh = i["x"] * r, i["dn"] * i["g"]
        dx = i["dres"] + r * (dxh - xh * (dxh * xh).mean(-1, keepdim=True))
        return {"n": xh * i["g"], "rstd": r[:, 0], "dx": dx, "dx16": dx,
                "dg": (i["dn"] * xh).sum(0)}
    if kind == "adam":
        i = {k: v.to(f64) for k, v in _adam_inputs(c, seed).items()}
        lr, b1, b2, eps, wd, t = ADAM_HP
        m = b1 * i["m"] + (1 - b1) * i["g"]
        v = b2 * i["v"] + (1 - b2) * i["g"].square()
        p = i["p"] * (1 - lr * wd) - lr / (1 - b1 ** t) * m / (
            v.sqrt() / math.sqrt(1 - b2 ** t) + eps)
        return {"p": p, "m": m, "v": v, "out": p}
    i = _acc_inputs(c, seed)
    return i["a"].to(f64) + i["g"].to(f64)
