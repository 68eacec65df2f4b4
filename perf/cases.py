"""The attention workloads whose speed is measured, with their inputs, the work they
cannot do without, and float64 results to compare with.

A case's ``kind`` names the entry point it goes through:

* ``train``  -- ``attention`` under autograd, forward and backward, on q, k, v tensors;
* ``packed`` -- ``attention_packed`` under autograd on one fused QKV projection;
* ``layer``  -- the ``MultiheadAttention`` module, forward and backward to its weights;
* ``fwd``    -- ``attention_fwd`` for inference: no log-sum-exp, prefill and decode.

Inputs are N(0, 1), as in the paper's measurements.
"""
from __future__ import annotations

import math

import torch

from paper_2112_05682_amd import attention, attention_fwd, attention_packed
from paper_2112_05682_amd.nn import MultiheadAttention

DTYPES = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"fp32": 4, "fp16": 2, "bf16": 2}


def _case(kind, dtype, B, H, n_q, n_k, d, d_v=None, causal=False, out_f32=False, kv_min=0, **more):
    """``kv_min``: 0 for no key padding, else the batches' valid key lengths run
    evenly from kv_min to n_k."""
    return {"kind": kind, "dtype": dtype, "B": B, "H": H, "n_q": n_q, "n_k": n_k, "d": d,
            "d_v": d if d_v is None else d_v, "causal": causal, "out_f32": out_f32, "kv_min": kv_min, **more}


def listed():
    return [
        # The paper's sweep starts at one head of 2^8 positions: here latency and launches count.
        _case("train", "fp32", 1, 1, 256, 256, 64, name="sweep_fp32_n256"),
        # The middle of that sweep in the paper's precision, 16-bit inputs and a float32 output.
        _case("train", "bf16", 1, 1, 4096, 4096, 64, out_f32=True, name="sweep_bf16_n4096"),
        # Training in float32: a small model that is checked or fine-tuned at full precision.
        _case("train", "fp32", 2, 8, 1000, 1000, 64, causal=True, name="train_fp32_causal_n1000"),
        # The benchmark's headline: long self-attention, forward and backward.
        _case("train", "bf16", 1, 16, 16384, 16384, 64, name="train_bf16_n16384"),
        # A causal language model's attention at a long context, the largest case.
        _case("train", "bf16", 4, 32, 8192, 8192, 128, causal=True, name="train_bf16_causal_n8192_d128"),
        # Cross-attention with narrower values: odd lengths, d_v != d.
        _case("train", "bf16", 2, 8, 700, 3001, 128, d_v=64, name="cross_bf16_dv64"),
        # A batch of padded sequences through an encoder's packed projection.
        _case("packed", "fp16", 16, 12, 512, 512, 64, kv_min=130, name="packed_fp16_padded_n512"),
        # One attention layer of a small language model in a training step.
        _case("layer", "bf16", 8, 8, 1024, 1024, 64, causal=True, name="layer_bf16_causal_n1024"),
        # One head against 2^20 keys, the end of the paper's sweep.
        _case("fwd", "bf16", 1, 1, 16384, 1 << 20, 64, name="longkv_bf16_nk1048576"),
        # Prefill of one prompt.
        _case("fwd", "bf16", 1, 32, 2047, 2047, 128, causal=True, name="prefill_bf16_n2047_d128"),
        # Decode: one query per sequence against a long cache.
        _case("fwd", "bf16", 8, 16, 1, 65536, 64, name="decode_bf16_nk65536"),
        # Decode of a few speculative tokens against caches of different lengths.
        _case("fwd", "fp16", 4, 32, 5, 7001, 128, kv_min=900, name="decode_fp16_padded_nk7001_d128"),
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["train"] * 5 + ["packed", "layer", "fwd", "fwd", "decode", "decode"])
    d = rng.choice([64, 64, 128])
    B, H = _log_uniform(rng, 1, 16), _log_uniform(rng, 1, 32)
    causal = rng.random() < 0.5
    if kind == "decode":
        n_q, n_k = rng.choice([1, 1, rng.randint(2, 64)]), _log_uniform(rng, 256, 1 << 17)
        while B * H * n_k * d > 1 << 31:
            n_k //= 2
        c = _case("fwd", rng.choice(["bf16", "fp16"]), B, H, n_q, n_k, d)
    elif kind == "fwd":
        n = _log_uniform(rng, 65, 16384)
        n_k = n if causal else rng.choice([n, _log_uniform(rng, 65, 1 << 18)])
        c = _case("fwd", rng.choice(["bf16", "bf16", "fp16", "fp32"]), B, H, n, n_k, d, causal=causal)
    elif kind == "train":
        dtype = rng.choice(["bf16", "bf16", "fp16", "fp32"])
        n = _log_uniform(rng, 100, 16384)
        n_k = n if causal else rng.choice([n, n, _log_uniform(rng, 100, 16384)])
        c = _case("train", dtype, B, H, n, n_k, d, d_v=rng.choice([d, d, d, 192 - d]), causal=causal,
                  out_f32=dtype != "fp32" and rng.random() < 0.25)
    else:
        n = _log_uniform(rng, 100, 4096)
        H = rng.choice([2, 4, 8, 12, 16])
        c = _case(kind, rng.choice(["bf16", "fp16"]), B, H, n, n, d, causal=causal)
    if c["B"] > 1 and c["kind"] != "train" and rng.random() < 0.4:
        c["kv_min"] = max(1, c["n_k"] // rng.randint(2, 8))
    # No dearer than the largest listed case; float32 products run at a sixteenth of the 16-bit rate.
    limit = 7e12 / (16 if c["dtype"] == "fp32" else 1)
    while work(c)["flops"] > limit:
        c["n_q"], c["n_k"] = max(65, c["n_q"] * 2 // 3), max(65, c["n_k"] * 2 // 3)
        c["kv_min"] = min(c["kv_min"], c["n_k"])
    return c


def _kv_lens(case):
    B, n, lo = case["B"], case["n_k"], case["kv_min"]
    return [n] * B if not lo else [lo + (n - lo) * b // max(1, B - 1) for b in range(B)]


def _pairs(case):
    """Query-key pairs that contribute to a pass."""
    n_q, total = case["n_q"], 0
    for n in _kv_lens(case):
        if case["causal"]:
            m = min(n_q, n)
            total += m * (m + 1) // 2 + (n_q - m) * n
        else:
            total += n_q * n
    return total * case["H"]


def work(case):
    B, H, n_q, n_k, d, dv = (case[x] for x in ("B", "H", "n_q", "n_k", "d", "d_v"))
    e, eo = BYTES[case["dtype"]], 4 if case["out_f32"] else BYTES[case["dtype"]]
    P = _pairs(case)
    keys = sum(min(n, n_q) if case["causal"] else n for n in _kv_lens(case)) * H
    qkv = e * (B * H * n_q * d + keys * (d + dv))
    o = eo * B * H * n_q * dv
    if case["kind"] == "fwd":
        return {"bytes": qkv + o, "flops": 2 * (d + dv) * P}
    # forward S, O; backward S again (the score matrix is never stored), dP, dV, dK, dQ
    flops = 2 * (d + dv) * P + 2 * (3 * d + 2 * dv) * P
    grads = e * B * H * (n_q * d + n_k * (d + dv))
    if case["kind"] != "layer":
        return {"bytes": qkv + 2 * o + grads, "flops": flops}
    E = H * d
    # x, dout, out, dx; the four projections' weights and their gradients
    return {"bytes": e * (4 * B * n_q * E + 2 * 4 * E * E), "flops": flops + 3 * 2 * B * n_q * 4 * E * E}


def tolerance(case):
    if case["dtype"] == "fp32":
        return {"rel": 1e-5}
    return {"rel": 1.6e-2 if case["dtype"] == "bf16" else 2e-3}


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    B, H, n_q, n_k, d, dv = (case[x] for x in ("B", "H", "n_q", "n_k", "d", "d_v"))
    dt = DTYPES[case["dtype"]]

    def normal(*shape, dtype=dt, std=1.0):
        return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * std).to(dtype)

    s = {"case": case, "kv_len": None}
    if case["kv_min"]:
        lens = torch.tensor(_kv_lens(case), dtype=torch.int32, device="cuda")
        s["kv_len"] = lens[torch.randperm(B, generator=g, device="cuda")].contiguous()
    if case["kind"] == "packed":
        s["qkv"] = normal(B, n_q, 3, H, d).requires_grad_()
        s["do"] = normal(B, n_q, H, d)
    elif case["kind"] == "layer":
        E = H * d
        m = MultiheadAttention(E, H, causal=case["causal"], device="cuda", dtype=dt)
        with torch.no_grad():
            for w in (m.qkv, m.out):
                w.weight.copy_(normal(*w.weight.shape, std=E ** -0.5))
                w.bias.copy_(normal(*w.bias.shape, std=0.02))
        s["module"], s["x"], s["do"] = m, normal(B, n_q, E).requires_grad_(), normal(B, n_q, E)
    else:
        s["q"], s["k"], s["v"] = normal(B, H, n_q, d), normal(B, H, n_k, d), normal(B, H, n_k, dv)
        if case["kind"] == "train":
            for x in ("q", "k", "v"):
                s[x].requires_grad_()
            s["do"] = normal(B, H, n_q, dv, dtype=torch.float32 if case["out_f32"] else dt)
    return s


def run(state):
    case, kv_len, causal = state["case"], state["kv_len"], state["case"]["causal"]
    if case["kind"] == "fwd":
        o, _ = attention_fwd(state["q"], state["k"], state["v"], causal=causal, need_lse=False, kv_len=kv_len)
        return {"o": o}
    if case["kind"] == "packed":
        o = attention_packed(state["qkv"], causal=causal, kv_len=kv_len)
        dqkv, = torch.autograd.grad(o, state["qkv"], state["do"])
        return {"o": o, "dqkv": dqkv}
    if case["kind"] == "layer":
        m = state["module"]
        out = m(state["x"], kv_len)
        grads = torch.autograd.grad(out, (state["x"], m.qkv.weight, m.qkv.bias, m.out.weight, m.out.bias), state["do"])
        return dict(zip(("o", "dx", "dw_qkv", "db_qkv", "dw_out", "db_out"), (out, *grads)))
    q, k, v = state["q"], state["k"], state["v"]
    o = attention(q, k, v, causal=causal, out_dtype=torch.float32 if case["out_f32"] else None, kv_len=kv_len)
    dq, dk, dv = torch.autograd.grad(o, (q, k, v), state["do"])
    return {"o": o, "dq": dq, "dk": dk, "dv": dv}


def _exact_attention(q, k, v, do, causal, kv_len):
    """Softmax attention of [B, H, n, features] float64 tensors and its gradients
    (None without ``do``), one (batch, head) and one block of query rows at a time."""
    B, H, n_q, d = q.shape
    n_k, scale = k.shape[2], 1.0 / math.sqrt(d)
    o = torch.zeros(B, H, n_q, v.shape[3], dtype=torch.float64, device=q.device)
    dq, dk, dv = (torch.zeros_like(t) for t in (q, k, v)) if do is not None else (None, None, None)
    for b in range(B):
        n = n_k if kv_len is None else int(kv_len[b])
        for h in range(H):
            kt, vt = k[b, h, :n], v[b, h, :n]
            step = max(1, (1 << 26) // n)
            for i in range(0, n_q, step):
                j = min(n_q, i + step)
                s = torch.mm(q[b, h, i:j], kt.t()).mul_(scale)
                if causal:
                    row = torch.arange(i, j, device=q.device)[:, None]
                    s.masked_fill_(torch.arange(n, device=q.device)[None, :] > row, -math.inf)
                p = torch.softmax(s, dim=1)
                o[b, h, i:j] = torch.mm(p, vt)
                if do is None:
                    continue
                g = do[b, h, i:j]
                dv[b, h, :n] += torch.mm(p.t(), g)
                ds = torch.mm(g, vt.t())
                ds.sub_((ds * p).sum(1, keepdim=True)).mul_(p)
                dq[b, h, i:j] = torch.mm(ds, kt).mul_(scale)
                dk[b, h, :n] += torch.mm(ds.t(), q[b, h, i:j]).mul_(scale)
    return o, dq, dk, dv


def exact(case, seed):
    s = prepare(case, seed)
    causal, lens = case["causal"], None if s["kv_len"] is None else s["kv_len"].tolist()
    with torch.no_grad():
        if case["kind"] == "layer":
            B, n, H, d = case["B"], case["n_q"], case["H"], case["d"]
            x, g = (s[t].double().reshape(B * n, H * d) for t in ("x", "do"))
            wi, bi, wo, bo = (t.double() for t in (s["module"].qkv.weight, s["module"].qkv.bias,
                                                   s["module"].out.weight, s["module"].out.bias))
            qkv = (torch.mm(x, wi.t()) + bi).view(B, n, 3, H, d)
            da = torch.mm(g, wo).view(B, n, H, d).transpose(1, 2)
        elif case["kind"] == "packed":
            qkv, da = s["qkv"].double(), s["do"].double().transpose(1, 2)
        if case["kind"] in ("layer", "packed"):
            q, k, v = (qkv[:, :, i].transpose(1, 2) for i in range(3))
        else:
            q, k, v = (s[t].double() for t in ("q", "k", "v"))
            da = s["do"].double() if "do" in s else None
        o, dq, dk, dv = _exact_attention(q, k, v, da, causal, lens)
        if case["kind"] == "fwd":
            return {"o": o}
        if case["kind"] == "train":
            return {"o": o, "dq": dq, "dk": dk, "dv": dv}
        dqkv = torch.stack([t.transpose(1, 2) for t in (dq, dk, dv)], dim=2)
        if case["kind"] == "packed":
            return {"o": o.transpose(1, 2), "dqkv": dqkv}
        a = o.transpose(1, 2).reshape(B * n, H * d)
        dqkv = dqkv.reshape(B * n, 3 * H * d)
        return {"o": (torch.mm(a, wo.t()) + bo).view(B, n, H * d), "dx": torch.mm(dqkv, wi).view(B, n, H * d),
                "dw_qkv": torch.mm(dqkv.t(), x), "db_qkv": dqkv.sum(0), "dw_out": torch.mm(g.t(), a),
                "db_out": g.sum(0)}
