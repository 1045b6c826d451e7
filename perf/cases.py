"""The attention and GEMM calls that this library's speed is judged by.

A case is one call of a public entry point (``attn_fwd``, ``attn_decode``,
``attn_decode_noalloc`` or ``gemm``) at one size, with the options it is
called with.  ``listed()`` holds twelve of them, from the launch-bound single
head to the largest prefill and GEMM; ``draw(rng)`` gives others of the same
ranges.  The exact results are the definitions in float64 torch.
"""
from __future__ import annotations

import math

import torch

import paper_2609_29219_amd as pa

DEV = "cuda"
# no drawn case does more than the largest listed ones
MAX_FLOPS = 1.0995e12
MAX_BYTES = 2.15e9


def _prefill(name, B, Hq, Hkv, Sq, Skv, d, causal, out, lse=False, mag=1.0):
    return {"name": name, "op": "prefill", "B": B, "Hq": Hq, "Hkv": Hkv, "Sq": Sq, "Skv": Skv,
            "d": d, "causal": causal, "out": out, "lse": lse, "mag": mag}


def _decode(name, B, Hq, Hkv, Skv, d, lse=False, noalloc=False):
    return {"name": name, "op": "decode", "B": B, "Hq": Hq, "Hkv": Hkv, "Skv": Skv, "d": d,
            "lse": lse, "noalloc": noalloc}


def _gemm(name, M, N, K, b_nk, out):
    return {"name": name, "op": "gemm", "M": M, "N": N, "K": K, "b_nk": b_nk, "out": out}


def listed():
    return [
        # one short head of an encoder-sized model: a call as small as any,
        # bound by the host path and the launch
        _prefill("prefill_single_head", 1, 1, 1, 256, 256, 64, False, "fp32"),
        # a batch of prompts, causal, equal query and key/value heads
        _prefill("prefill_causal", 4, 16, 16, 2048, 2048, 128, True, "fp32"),
        # one long sequence without a mask: the largest prefill
        _prefill("prefill_long", 1, 32, 32, 8192, 8192, 128, False, "fp32", mag=0.5),
        # prompts of a grouped-query model whose length is no multiple of any
        # tile, bf16 output, with the log-sum-exp that a later merge needs
        _prefill("prefill_gqa_ragged", 2, 32, 8, 1777, 1777, 128, True, "bf16", lse=True),
        # chunked prefill: 512 new tokens against a 16k key/value cache
        _prefill("prefill_chunk", 1, 32, 8, 512, 16384, 128, True, "bf16"),
        # 64-dimensional heads, no mask (an encoder batch)
        _prefill("prefill_d64", 4, 16, 16, 2048, 2048, 64, False, "fp32"),
        # one token for each of 16 sequences, every query head with its own
        # keys and values: the largest decode
        _decode("decode_batch", 16, 32, 32, 8192, 128),
        # a grouped-query model's decode batch at an odd cache length
        _decode("decode_gqa", 8, 64, 8, 4099, 128, lse=True),
        # one token of one short sequence through the entry point that does
        # not allocate: the smallest decode
        _decode("decode_small", 1, 32, 8, 777, 128, noalloc=True),
        # a large square product: the largest GEMM
        _gemm("gemm_square", 8192, 8192, 8192, False, "fp32"),
        # a tall product with few columns (the skewed shapes)
        _gemm("gemm_tall", 16384, 256, 2048, False, "fp32"),
        # a linear layer (weights stored [out][in]) over a small batch of
        # tokens that fills no tile
        _gemm("gemm_few_rows", 100, 4096, 4096, True, "bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_any(rng):
    op = rng.choice(["prefill", "prefill", "decode", "gemm"])
    if op == "gemm":
        # K and N in the multiples of 8 that the entry point takes
        return _gemm("", _log(rng, 64, 16384), 8 * _log(rng, 32, 2048), 8 * _log(rng, 32, 2048),
                     rng.random() < 0.5, rng.choice(["fp32", "bf16"]))
    d = rng.choice([64, 128, 128])
    Hkv, group = rng.choice([(1, 1), (1, 8), (2, 4), (4, 8), (8, 4), (8, 8), (16, 1), (16, 2),
                             (32, 1)])
    if op == "decode":
        return _decode("", rng.choice([1, 1, 2, 4, 8, 16, 32]), Hkv * group, Hkv,
                       _log(rng, 300, 131072), d, rng.random() < 0.5, rng.random() < 0.3)
    causal = rng.random() < 0.5
    if rng.random() < 0.3:  # a chunk of new tokens against a cache
        Sq = _log(rng, 16, 1024)
        Skv = Sq + _log(rng, 1024, 32768)
    else:
        Sq = Skv = _log(rng, 200, 8192)
    return _prefill("", rng.choice([1, 1, 2, 3, 4, 8]), Hkv * group, Hkv, Sq, Skv, d, causal,
                    rng.choice(["fp32", "bf16"]), rng.random() < 0.3, rng.choice([1.0, 0.5]))


def draw(rng):
    while True:
        case = _draw_any(rng)
        w = work(case)
        if w["flops"] > MAX_FLOPS or w["bytes"] > MAX_BYTES:
            continue
        if case["op"] == "decode" and case["noalloc"]:
            # that entry point's partials have to fit its fixed scratch; at
            # most 512 splits, one for each 128 keys
            splits = min(512, -(-case["Skv"] // 128))
            if case["B"] * case["Hq"] * splits * (case["d"] + 2) * 4 > pa.NOALLOC_SCRATCH_BYTES:
                continue
        del case["name"]
        return case


def _out_dtype(case):
    return torch.bfloat16 if case["out"] == "bf16" else torch.float32


def _randn(g, *shape, mag=1.0):
    # in pieces, so that the float32 draws of a large cache stay small
    t = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    flat = t.view(-1)
    step = 1 << 26
    for i in range(0, flat.numel(), step):
        n = min(step, flat.numel() - i)
        flat[i:i + n] = torch.randn(n, generator=g, device=DEV) * mag
    return t


def prepare(case, seed):
    """Unit-normal bf16 operands (queries, keys and values of a normalised
    layer, GEMM operands); ``mag`` scales them."""
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    if case["op"] == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        a = _randn(g, M, K)
        b = _randn(g, N, K) if case["b_nk"] else _randn(g, K, N)
        return {"case": case, "a": a, "b": b}
    B, Hq, Hkv, Skv, d = (case[n] for n in ("B", "Hq", "Hkv", "Skv", "d"))
    state = {"case": case}
    if case["op"] == "prefill":
        state["q"] = _randn(g, B, Hq, case["Sq"], d, mag=case["mag"])
    else:
        state["q"] = _randn(g, B, Hq, d)
    mag = case.get("mag", 1.0)
    state["k"] = _randn(g, B, Hkv, Skv, d, mag=mag)
    state["v"] = _randn(g, B, Hkv, Skv, d, mag=mag)
    if case["op"] == "decode" and case["noalloc"]:
        # buffers that such a caller holds from the start
        state["o"] = torch.empty((B, Hq, d), dtype=torch.float32, device=DEV)
        state["lse"] = (torch.empty((B, Hq), dtype=torch.float32, device=DEV)
                        if case["lse"] else None)
    return state


def run(state):
    case = state["case"]
    if case["op"] == "gemm":
        return pa.gemm(state["a"], state["b"], b_nk=case["b_nk"], out_dtype=_out_dtype(case))
    q, k, v = state["q"], state["k"], state["v"]
    if case["op"] == "prefill":
        return pa.attn_fwd(q, k, v, causal=case["causal"], out_dtype=_out_dtype(case),
                           return_lse=case["lse"])
    if case["noalloc"]:
        o = pa.attn_decode_noalloc(q, k, v, state["o"], lse=state["lse"])
        return (o, state["lse"]) if case["lse"] else o
    return pa.attn_decode(q, k, v, return_lse=case["lse"])


def work(case):
    """bf16 operands read once, results written once; 4 d operations for each
    (query, key) pair that the mask allows, 2 for each product of the GEMM."""
    if case["op"] == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        out = 2 if case["out"] == "bf16" else 4
        return {"bytes": 2 * (M * K + K * N) + out * M * N, "flops": 2 * M * N * K}
    B, Hq, Hkv, Skv, d = (case[n] for n in ("B", "Hq", "Hkv", "Skv", "d"))
    Sq = case.get("Sq", 1)
    out = 2 if case.get("out") == "bf16" else 4
    pairs = Sq * Skv
    if case.get("causal"):
        pairs -= Sq * (Sq - 1) // 2
    rows = B * Hq * Sq
    return {"bytes": rows * d * (2 + out) + 4 * B * Hkv * Skv * d + (4 * rows if case["lse"] else 0),
            "flops": 4 * d * pairs * B * Hq}


def tolerance(case):
    """About four times the relative error that the path shows against the
    exact result: bf16 probabilities in prefill (up to 2.3e-3 with a bf16
    output) and in decode for groups of 4 and more query heads (1.4e-3), fp32
    sums elsewhere (decode 4.4e-7, GEMM 5.7e-7 at K = 8192), one rounding of a
    bf16 GEMM output (1.7e-3)."""
    if case["op"] == "gemm":
        return {"rel": 7e-3} if case["out"] == "bf16" else {"rel": 5e-6}
    if case["op"] == "prefill":
        return {"rel": 1e-2}
    return {"rel": 6e-3} if case["Hq"] // case["Hkv"] >= 4 else {"rel": 5e-6}


def exact(case, seed):
    state = prepare(case, seed)
    if case["op"] == "gemm":
        a, b = state["a"].double(), state["b"].double()
        return a @ (b.t().contiguous() if case["b_nk"] else b)
    q, k, v = state["q"], state["k"], state["v"]
    B, Hq, Hkv, Skv, d = (case[n] for n in ("B", "Hq", "Hkv", "Skv", "d"))
    Sq = case.get("Sq", 1)
    group = Hq // Hkv
    scale = 1.0 / math.sqrt(d)
    q = q.view(B, Hkv, group * Sq, d)
    o = torch.empty((B, Hkv, group * Sq, d), dtype=torch.float64, device=DEV)
    lse = torch.empty((B, Hkv, group * Sq), dtype=torch.float64, device=DEV)
    keys = torch.arange(Skv, device=DEV)
    step = max(1, (1 << 26) // Skv)  # query rows whose scores are held at once
    for b in range(B):
        for h in range(Hkv):
            kt, vv = k[b, h].double().t().contiguous(), v[b, h].double()
            for r in range(0, group * Sq, step):
                rows = torch.arange(r, min(group * Sq, r + step), device=DEV)
                s = (q[b, h, r:r + step].double() @ kt) * scale
                if case.get("causal"):
                    last = rows % Sq + (Skv - Sq)
                    s.masked_fill_(keys[None, :] > last[:, None], -math.inf)
                z = torch.logsumexp(s, dim=-1)
                lse[b, h, r:r + step] = z
                o[b, h, r:r + step] = torch.exp(s - z[:, None]) @ vv
    shape = (B, Hq, Sq) if case["op"] == "prefill" else (B, Hq)
    o, lse = o.view(*shape, d), lse.view(*shape)
    return (o, lse) if case["lse"] else o
