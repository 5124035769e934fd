"""The work a user of this library has it do, as timed cases over its public entry points.

Three kinds of call, each the way an inference program makes it (weights, routing tables and
output buffers in hand, one pass through the package's functions on the current stream):

* ``dense``: one projection GEMM over block-quantised weights (``dense``), from a decode step's
  single row to a 2048-token prompt;
* ``moe``: one MoE feed-forward block over routed tokens (``moe_bucket``,
  ``moe_gate_up_swiglu``, ``moe_grouped``, ``moe_combine``), from a decode batch to a long prompt;
* ``attn``: one prefill attention layer (``attention_prefill``).

Inputs follow the distributions of the workloads in ``synth``: activations N(0, 1) in bf16, Q8
weights uniform in [-127, 127] with scales in [0.001, 0.01], Q4 nibbles uniform with scales in
[0.005, 0.02], router logits N(0, 1) (plus ``-skew * ln(e + 1)`` for expert e), top-k of the softmax,
renormalised weights; attention q, k and v N(0, 1).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2607_19438_amd as qg

FORMATS = {"q8": qg.Q8, "q4": qg.Q4}
SCALES = {"q8": (0.001, 0.01), "q4": (0.005, 0.02)}


def _dense(name, fmt, M, N, K):
    return {"name": name, "kind": "dense", "fmt": fmt, "M": M, "N": N, "K": K}


def _moe(name, fmt, T, E, topk, hidden, inter, skew):
    return {"name": name, "kind": "moe", "fmt": fmt, "T": T, "E": E, "topk": topk, "hidden": hidden, "inter": inter,
            "skew": skew}


def _attn(name, B, S, H, Hkv, D, causal):
    return {"name": name, "kind": "attn", "B": B, "S": S, "H": H, "Hkv": Hkv, "D": D, "causal": causal}


def listed():
    return [
        # one decode step's up projection: the smallest call, one row against 17 MB of weights
        _dense("dense_q8_m1", "q8", 1, 8192, 2048),
        # verification of five drafted tokens through a down projection (few weight rows, long K)
        _dense("dense_q4_m5", "q4", 5, 2048, 8192),
        # a short prompt's projection with a small hidden size: launch latency
        _dense("dense_q8_m128", "q8", 128, 1024, 1024),
        # a medium prompt through a 4-bit up projection
        _dense("dense_q4_m512", "q4", 512, 8192, 3072),
        # a 2048-token prompt through the gate/up and the down projection of an 8-bit model
        _dense("dense_q8_gate_up", "q8", 2048, 8192, 2048),
        _dense("dense_q8_down", "q8", 2048, 2048, 8192),
        # MoE feed-forward block of a decode batch: one to a few rows per active expert
        _moe("moe_q4_t4", "q4", 4, 128, 8, 2048, 768, 0.0),
        # a short prompt with skewed routing: about half of the experts active, most with few rows
        _moe("moe_q4_t128", "q4", 128, 128, 8, 2048, 768, 1.2),
        # an odd prompt length through an 8-bit MoE with fewer experts and an odd inner size
        _moe("moe_q8_t777", "q8", 777, 64, 6, 2048, 1056, 0.0),
        # a 2048-token prompt, experts evenly loaded
        _moe("moe_q4_t2048", "q4", 2048, 128, 8, 2048, 768, 0.0),
        # a long prompt with skewed routing: groups from none to thousands of rows
        _moe("moe_q4_t8192", "q4", 8192, 128, 8, 2048, 768, 1.2),
        # the attention layer of a 2048-token prompt, grouped-query heads
        _attn("attn_s2048", 1, 2048, 32, 4, 128, True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["dense", "dense", "moe", "moe", "attn"])
    if kind == "dense":
        M = _log_uniform(rng, 1, 2048)
        N = _log_uniform(rng, 256, 8192)
        if rng.random() < 0.5:
            N = N // 64 * 64
        K = 32 * _log_uniform(rng, 16, 256)
        return {"kind": kind, "fmt": rng.choice(["q8", "q4"]), "M": M, "N": N, "K": K}
    if kind == "moe":
        E = rng.choice([8, 32, 64, 96, 128])
        topk = rng.choice([k for k in (1, 2, 4, 6, 8) if k <= E // 2])
        T = _log_uniform(rng, 1, 8192)
        hidden = 64 * rng.randint(8, 32)
        inter = 32 * rng.randint(8, 24)
        return {"kind": kind, "fmt": rng.choice(["q8", "q4"]), "T": T, "E": E, "topk": topk, "hidden": hidden,
                "inter": inter, "skew": rng.choice([0.0, 0.0, 0.6, 1.2])}
    S = _log_uniform(rng, 64, 4096)
    H, Hkv = rng.choice([(8, 8), (16, 4), (32, 4), (32, 8)])
    B = rng.randint(1, 4) if S <= 1024 else 1
    return {"kind": kind, "B": B, "S": S, "H": H, "Hkv": Hkv, "D": rng.choice([64, 128]), "causal": rng.random() < 0.7}


def _weights(gen, shape, K, fmt):
    """Packed weights [*shape][K or K/2] and fp16 scales [*shape][K/32]."""
    lo, hi = SCALES[fmt]
    if fmt == "q8":
        wq = torch.randint(-127, 128, (*shape, K), dtype=torch.int8, device="cuda", generator=gen)
    else:
        wq = torch.randint(0, 256, (*shape, K // 2), dtype=torch.uint8, device="cuda", generator=gen)
    scales = torch.empty((*shape, K // 32), dtype=torch.float32, device="cuda").uniform_(lo, hi, generator=gen)
    return wq, scales.to(torch.float16)


def _inputs(case, seed):
    """The tensors of one call, from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(*shape):
        return torch.randn(shape, dtype=torch.float32, device="cuda", generator=gen).to(torch.bfloat16)

    if case["kind"] == "dense":
        x = normal(case["M"], case["K"])
        wq, scales = _weights(gen, (case["N"],), case["K"], case["fmt"])
        return {"x": x, "wq": wq, "scales": scales}
    if case["kind"] == "moe":
        T, E, topk, hidden, inter = (case[k] for k in ("T", "E", "topk", "hidden", "inter"))
        x = normal(T, hidden)
        logits = torch.randn((T, E), dtype=torch.float32, device="cuda", generator=gen)
        logits -= case["skew"] * torch.log(torch.arange(1, E + 1, dtype=torch.float32, device="cuda"))
        p, idx = torch.topk(torch.softmax(logits, dim=1), topk, dim=1)
        route_w = (p / p.sum(dim=1, keepdim=True)).reshape(-1).contiguous()
        idx = idx.reshape(-1).to(torch.int32)
        counts = torch.bincount(idx, minlength=E)
        offsets = torch.zeros(E + 1, dtype=torch.int32, device="cuda")
        offsets[1:] = torch.cumsum(counts, 0)
        return {"x": x, "idx": idx, "offsets": offsets, "route_w": route_w,
                "gate_up": _weights(gen, (E, 2 * inter), hidden, case["fmt"]),
                "down": _weights(gen, (E, hidden), inter, case["fmt"])}
    B, S, H, Hkv, D = (case[k] for k in ("B", "S", "H", "Hkv", "D"))
    return {"q": normal(B, S, H, D), "k": normal(B, S, Hkv, D), "v": normal(B, S, Hkv, D)}


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case

    def buf(*shape, dtype=torch.float32):
        return torch.empty(shape, dtype=dtype, device="cuda")

    if case["kind"] == "dense":
        s["y"] = buf(case["M"], case["N"])
    elif case["kind"] == "moe":
        T, topk, hidden, inter = (case[k] for k in ("T", "topk", "hidden", "inter"))
        fmt = FORMATS[case["fmt"]]
        s["gate_up"] = qg.ExpertTable(*s["gate_up"], fmt)
        s["down"] = qg.ExpertTable(*s["down"], fmt)
        s["perm"] = buf(T * topk, dtype=torch.int32)
        s["h"] = buf(T * topk, inter, dtype=torch.bfloat16)
        s["y2"] = buf(T * topk, hidden)
        s["out"] = buf(T, hidden)
    else:
        s["o"] = torch.empty_like(s["q"])
    return s


def run(state):
    case = state["case"]
    if case["kind"] == "dense":
        return qg.dense(state["x"], state["wq"], state["scales"], FORMATS[case["fmt"]], out=state["y"])
    if case["kind"] == "moe":
        fmt, topk, offsets = FORMATS[case["fmt"]], case["topk"], state["offsets"]
        perm = qg.moe_bucket(state["idx"], offsets, out=state["perm"])
        h = qg.moe_gate_up_swiglu(state["x"], perm, offsets, state["gate_up"], None, topk, fmt, out=state["h"])
        y2 = qg.moe_grouped(h, perm, offsets, state["down"], None, 1, fmt, out=state["y2"])
        return qg.moe_combine(y2, state["route_w"], topk, out=state["out"])
    return qg.attention_prefill(state["q"], state["k"], state["v"], causal=case["causal"], out=state["o"])


def _weight_bytes(fmt, rows, K):
    return rows * K * (1.0 if fmt == "q8" else 0.5) + rows * K / 32 * 2


def _active_experts(case):
    """Experts that receive a token in one draw of the case's routing."""
    rng = np.random.default_rng(0)
    logits = rng.standard_normal((case["T"], case["E"])) - case["skew"] * np.log(np.arange(1, case["E"] + 1))
    return len(np.unique(np.argsort(-logits, axis=1)[:, :case["topk"]]))


def work(case):
    if case["kind"] == "dense":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": M * K * 2 + _weight_bytes(case["fmt"], N, K) + M * N * 4, "flops": 2.0 * M * N * K}
    if case["kind"] == "moe":
        T, topk, hidden, inter = (case[k] for k in ("T", "topk", "hidden", "inter"))
        per_expert = _weight_bytes(case["fmt"], 2 * inter, hidden) + _weight_bytes(case["fmt"], hidden, inter)
        return {"bytes": T * hidden * 2 + _active_experts(case) * per_expert + T * topk * 8 + T * hidden * 4,
                "flops": 2.0 * T * topk * 3 * inter * hidden}
    B, S, H, Hkv, D = (case[k] for k in ("B", "S", "H", "Hkv", "D"))
    pairs = S * (S + 1) // 2 if case["causal"] else S * S
    return {"bytes": 2.0 * B * S * D * (2 * H + 2 * Hkv), "flops": 4.0 * B * H * D * pairs}


def tolerance(case):
    # about four times the measured distance from the 64-bit result (dense 1.7e-3, moe 3.3e-3, attn
    # 2.0e-3): the bf16 rounding of the weights (dense), of the weights and of the gated activations
    # between the projections (moe), of the softmax weights and of the output (attn)
    return {"rel": {"dense": 7e-3, "moe": 1.3e-2, "attn": 8e-3}[case["kind"]]}


def _dequantise(wq, scales, fmt):
    """float64 [N][K] of one packed weight matrix."""
    if fmt == "q8":
        q = wq.to(torch.float64)
    else:
        q = torch.stack((wq & 15, wq >> 4), dim=-1).reshape(wq.shape[0], -1).to(torch.float64) - 8.0
    return q * scales.to(torch.float64).repeat_interleave(32, dim=1)


def exact(case, seed):
    s = _inputs(case, seed)
    if case["kind"] == "dense":
        return s["x"].to(torch.float64) @ _dequantise(s["wq"], s["scales"], case["fmt"]).t().contiguous()
    if case["kind"] == "moe":
        T, E, topk, inter = (case[k] for k in ("T", "E", "topk", "inter"))
        x = s["x"].to(torch.float64)
        idx = s["idx"].to(torch.int64)
        out = torch.zeros((T, case["hidden"]), dtype=torch.float64, device="cuda")
        for e in range(E):
            slots = torch.nonzero(idx == e).reshape(-1)
            if slots.numel() == 0:
                continue
            w1 = _dequantise(s["gate_up"][0][e], s["gate_up"][1][e], case["fmt"]).t().contiguous()
            w2 = _dequantise(s["down"][0][e], s["down"][1][e], case["fmt"]).t().contiguous()
            y1 = x[slots // topk] @ w1
            h = torch.nn.functional.silu(y1[:, :inter]) * y1[:, inter:]
            out.index_add_(0, slots // topk, (h @ w2) * s["route_w"][slots].to(torch.float64)[:, None])
        return out
    B, S, H, Hkv, D = (case[k] for k in ("B", "S", "H", "Hkv", "D"))
    out = torch.empty((B, S, H, D), dtype=torch.float64, device="cuda")
    mask = torch.ones((S, S), dtype=torch.bool, device="cuda").tril() if case["causal"] else None
    for b in range(B):
        for h in range(H):
            g = h // (H // Hkv)
            q, k, v = (s[n][b, :, i].to(torch.float64).contiguous() for n, i in (("q", h), ("k", g), ("v", g)))
            z = (q @ k.t().contiguous()) / math.sqrt(D)
            if mask is not None:
                z = z.masked_fill(~mask, float("-inf"))
            out[b, :, h] = torch.softmax(z, dim=1) @ v
    return out
