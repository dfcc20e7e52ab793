"""The cases this repository's speed is measured on: what they are, their inputs, one
pass of each through the public entry points, the work a pass cannot do without, and how
far the results of two correct implementations may differ.

A case is a dict of plain values.  Its "kind" is the call a user's program makes:

  decode    one step over a KV cache, every sequence of the same length
  ragged    one step over sequences of different lengths in one cache allocation
  prefill   the whole prefill of a prompt, block-mean summaries
  learned   the same with learned summary queries (the stage-level calls)
  append    a prompt continued against a longer cache (summaries of the new chunks,
            routing, attention)
  train     prefill that keeps its lists, then the backward pass

Inputs are those of paper_2605_18753_amd.inputs: N(0,1) tensors with an offset shared by
the keys of a chunk (or needle chunks), optionally with queries that vary smoothly along the
sequence, drawn on the GPU from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2605_18753_amd import binding as B
from paper_2605_18753_amd.inputs import Workload, make_inputs

DEV = "cuda:0"


def _case(kind, batch, h_q, h_kv, n_q, n_kv, d=128, block=64, **kw):
    c = dict(kind=kind, batch=batch, h_q=h_q, h_kv=h_kv, n_q=n_q, n_kv=n_kv, d=d, block=block, alpha=1.5, gamma=1.0,
             sigma=1.0, causal=True, window=0, dtype="bf16", offset=0.5, needles=0, corr=0.0)
    c.update(kw)
    return c


def listed():
    return [
        # one sequence at the start of its answer: nothing but latency and launches
        dict(_case("decode", 1, 32, 8, 1, 1000, offset=0.7), name="decode_1k"),
        # the decode point of the paper's kernel benchmark (batch 24, GQA group 16, 32k, a quarter of
        # the chunks kept), prior strength of its trained models
        dict(_case("decode", 24, 32, 2, 1, 32768, gamma=3.0, sigma=1e6), name="decode_32k_g16"),
        # the 128k decode configuration at the temperature that keeps a quarter of the chunks
        dict(_case("decode", 16, 32, 8, 1, 131072, gamma=0.4, offset=0.7), name="decode_128k"),
        # a serving batch: lengths between a quarter of the cache and all of it, the last
        # block always attended
        dict(_case("ragged", 12, 32, 8, 1, 20000, window=1, sigma=1e6, offset=0.7), name="ragged_20k"),
        # a chat turn of odd length
        dict(_case("prefill", 1, 32, 8, 1000, 1000), name="prefill_1k"),
        # a prompt of the paper's benchmark shape with learned summaries, the local window and
        # the prior strength of the trained models, neighbouring tokens with similar queries
        dict(_case("learned", 1, 32, 2, 16384, 16384, gamma=2.5, sigma=1e6, window=1, corr=0.97), name="learned_16k_g16"),
        # the headline configuration: 32k causal GQA prefill
        dict(_case("prefill", 1, 32, 8, 32768, 32768), name="prefill_32k"),
        # the long prefill, 128k tokens in chunks of 128
        dict(_case("prefill", 1, 32, 8, 131072, 131072, block=128, offset=1.0), name="prefill_128k"),
        # a piece of a long prompt (chunked prefill) of odd length against the cache before it
        dict(_case("append", 1, 32, 8, 2000, 32720, gamma=1.5, corr=0.9), name="append_2k_to_32k"),
        # the training-shaped configuration, forward and backward
        dict(_case("train", 4, 16, 16, 8192, 8192, sigma=1e6, offset=0.0, needles=4), name="train_8k"),
        # training of a small grouped-query model: odd length, head dimension 64
        dict(_case("train", 2, 16, 4, 3001, 3001, d=64, sigma=1e6, offset=0.8), name="train_3k_d64"),
        # the fp32 single-head configuration, forward and backward
        dict(_case("train", 1, 1, 1, 1024, 1024, d=64, sigma=1e6, causal=False, dtype="fp32"), name="fp32_1k"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "ragged", "prefill", "prefill", "learned", "append", "train", "train", "fp32"])
    d = rng.choice([128, 128, 128, 64])
    block = rng.choice([64, 64, 64, 128])
    h_kv = rng.choice([1, 2, 4, 8])
    g = rng.choice([1, 2, 4, 4, 8, 16])
    while h_kv * g > 32:
        g //= 2
    # a chunk is kept if one head keeps it: larger groups need sharper scores for the same sparsity
    kw = dict(alpha=rng.choice([1.5, 1.5, 1.5, 1.25, 2.0]), gamma=round(rng.uniform(0.4, 3.0 if g >= 8 else 1.5), 2),
              sigma=rng.choice([1.0, 10.0, 1e6]), window=rng.choice([0, 0, 1]), offset=round(rng.uniform(0.4, 0.8), 2))
    if kind in ("decode", "ragged"):
        n = _log_int(rng, 500, 131072)
        # caches of up to 2^31 elements, as in the listed 128k step
        top = max(1, min(32, (1 << 31) // (n * d * h_kv)))
        return _case(kind, _log_int(rng, 1, top), h_kv * g, h_kv, 1, n, d, block, **kw)
    if kind in ("prefill", "learned"):
        n = _log_int(rng, 300, 50000)
        return _case(kind, rng.choice([1, 2]) if n < 8192 else 1, h_kv * g, h_kv, n, n, d, block,
                     corr=rng.choice([0.0, 0.9, 0.97]), **kw)
    if kind == "append":
        # the cache before the new tokens is a multiple of 64 tokens
        old, n = 64 * _log_int(rng, 16, 900), _log_int(rng, 65, 4096)
        return _case(kind, 1, h_kv * g, h_kv, n, old + n, d, block, corr=rng.choice([0.0, 0.9, 0.97]), **kw)
    # Gradients at the prior strength of the trained models: at sigma = 1 the gradient of a
    # chunk at the edge of its support is unbounded (1/w), and the norm of the whole gradient is
    # that of the few rows nearest to the edge, on which no two correct implementations agree.
    kw["sigma"] = 1e6
    if kind == "train":
        n = _log_int(rng, 300, 12000)
        return _case(kind, rng.choice([1, 2, 4]) if n < 4096 else 1, h_kv * g, h_kv, n, n, d, block, **kw)
    n = _log_int(rng, 4, 32) * 64 + rng.randrange(0, 64)
    causal = rng.random() < 0.5
    if not causal:
        n, kw["window"] = n // block * block, 0
    return _case("train", 1, g, 1, n, n, d, block, causal=causal, dtype="fp32", **kw)


def prepare(case, seed):
    c = case
    w = Workload("case", c["batch"], c["h_q"], c["h_kv"], c["n_q"], c["n_kv"], c["d"], c["block"], causal=c["causal"],
                 dtype=c["dtype"], offset_sigma=c["offset"], needles=c["needles"], query_corr=c["corr"], seed=seed)
    q, k, v = make_inputs(w, DEV)
    o = torch.empty_like(q)
    p = B.make_params(q, k, v, o, c["block"], c["alpha"], c["gamma"], c["sigma"], c["causal"], window=c["window"])
    s = dict(kind=c["kind"], p=p, q=q, k=k, v=v, o=o, ws=B.alloc_workspace(p, DEV), lists=B.Lists(),
             kbar=torch.empty(B.kbar_shape(p), dtype=torch.float32, device=DEV))
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed + 1)
    if c["kind"] in ("decode", "ragged", "append"):
        B.dash_kbar_compress(p, k, s["kbar"])          # the summary cache of the tokens so far
    if c["kind"] == "ragged":
        lens = torch.randint(max(1, c["n_kv"] // 4), c["n_kv"] + 1, (c["batch"],), generator=gen, device=DEV)
        s["lens"] = lens.to(torch.int32)
    if c["kind"] == "append":
        s["first"] = (c["n_kv"] - c["n_q"]) // c["block"]
        s["new"] = c["n_kv"] // c["block"] - s["first"]
    if c["kind"] == "learned":
        s["qbar"] = torch.randn((c["h_kv"], c["d"]), generator=gen, device=DEV, dtype=torch.float32)
    if c["kind"] == "train":
        s["d_o"] = torch.randn(q.shape, generator=gen, device=DEV, dtype=torch.float32).to(q.dtype)
        s["lists"] = B.Lists.allocate(p, DEV, idx=False)
        s["dq"], s["dk"], s["dv"] = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
        s["wsb"] = B.alloc_backward_workspace(p, DEV)
    return s


def run(s):
    p, q, k, v, o, kbar, lists, ws = s["p"], s["q"], s["k"], s["v"], s["o"], s["kbar"], s["lists"], s["ws"]
    kind = s["kind"]
    if kind == "decode":
        B.dash_attn_decode(p, q, k, v, kbar, o, lists, ws)
    elif kind == "ragged":
        B.dash_attn_decode_ragged(p, q, k, v, kbar, s["lens"], o, lists, ws)
    elif kind == "append":
        if s["new"] > 0:
            B.dash_kbar_compress(p, k, kbar, s["first"], s["new"])
        B.dash_stage1_route(p, q, kbar, lists, ws)
        B.dash_stage2_attend(p, q, k, v, o, lists, ws)
    elif kind == "learned":
        B.dash_kbar_summarize(p, k, s["qbar"], kbar)
        B.dash_stage1_route(p, q, kbar, lists, ws)
        B.dash_stage2_attend(p, q, k, v, o, lists, ws)
    else:
        B.dash_attn_prefill(p, q, k, v, o, kbar, lists, ws)
    if kind != "train":
        return {"o": o, "kbar": kbar}
    B.dash_attn_backward(p, q, k, v, s["d_o"], kbar, lists, s["dq"], s["dk"], s["dv"], s["wsb"])
    return {"o": o, "kbar": kbar, "mask": lists.mask, "tau": lists.tau, "dq": s["dq"], "dk": s["dk"], "dv": s["dv"]}


def _kept(case, n_cand, samples=8):
    """Routed chunks of a token with n_cand candidates, expected on these inputs: the scores
    of an independent query are N(0, s^2) with s = gamma (alpha - 1) sqrt(offset^2 + 1/block); a
    chunk is kept if one head of the group keeps it."""
    if n_cand <= 0:
        return 0.0
    a1 = case["alpha"] - 1.0
    g = case["h_q"] // case["h_kv"]
    std = case["gamma"] * a1 * math.sqrt((0.0 if case["needles"] else case["offset"]) ** 2 + 1.0 / case["block"])
    x = np.random.default_rng(n_cand).standard_normal((samples, g, n_cand)) * std
    hi = x.max(-1, keepdims=True)
    lo = hi - 1.0
    for _ in range(30):
        mid = 0.5 * (lo + hi)
        more = (np.maximum(x - mid, 0.0) ** (1.0 / a1)).sum(-1, keepdims=True) > 1.0
        lo, hi = np.where(more, mid, lo), np.where(more, hi, mid)
    return float((x > lo).any(1).sum(-1).mean())


def _attended(case):
    """(attended keys, candidate chunks) per query, averaged over the queries."""
    blk, n_kv, n_q = case["block"], case["n_kv"], case["n_q"]
    if case["kind"] == "ragged":
        ends = [n_kv // 4 + (n_kv - n_kv // 4) * (i + 0.5) / 8 for i in range(8)]
    else:
        steps = min(16, n_q)
        ends = [n_kv - n_q + n_q * (i + 0.5) / steps + 0.5 for i in range(steps)]
    keys = cand = 0.0
    for e in ends:
        e = max(1, min(n_kv, int(e)))
        if not case["causal"]:
            n = n_kv // blk
            keys, cand = keys + _kept(case, n) * blk, cand + n
            continue
        own = (e - 1) // blk
        n = max(own - case["window"], 0)
        keys += _kept(case, n) * blk + (own - n) * blk + (e - own * blk)
        cand += n
    return keys / len(ends), cand / len(ends)


def work(case):
    c = case
    es = 2 if c["dtype"] == "bf16" else 4
    keys, cand = _attended(c)
    rows = c["batch"] * c["h_q"] * c["n_q"]
    kbar = c["batch"] * c["h_kv"] * (c["n_kv"] // c["block"]) * c["d"] * 4
    q_bytes = rows * c["d"] * es
    kv_bytes = c["batch"] * c["h_kv"] * c["n_kv"] * c["d"] * es
    flops = rows * c["d"] * (4.0 * keys + 2.0 * cand)      # attention, routing scores
    if c["n_q"] == 1:
        # the attended keys and values, the summaries of the candidates
        pairs = c["batch"] * c["h_kv"]
        return {"bytes": 2.0 * q_bytes + pairs * c["d"] * (keys * 2 * es + cand * 4), "flops": flops}
    bytes_ = 2.0 * q_bytes + 2.0 * kv_bytes + kbar
    if c["kind"] == "train":
        # five products per attended pair against the forward's two; dO in; dq, dk, dv out
        flops += rows * c["d"] * 10.0 * keys
        bytes_ += 2.0 * q_bytes + 2.0 * kv_bytes
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # bf16: one rounding of the results and of the P operand.  fp32: sums of up to a few thousand
    # terms in any order.  A chunk exactly at its threshold may fall on either side of it, which
    # moves its row (and its mask bit) and no other.
    if case["dtype"] == "fp32":
        return {"rel": 5e-5, "max": 5e-3, "differ": 1e-4}
    return {"rel": 1e-2, "max": 0.4, "differ": 1e-4}
