"""The work a provider node has this library do, as cases that can be timed one by one.

A node's requests reach the library as www_prefill calls (whole prompts, or chunks over a cached prefix), as
www_decode_step calls (one token for every running sequence) and, for sampled generation, as www_sample_top_p calls.  The
listed cases span the model shapes, batch sizes, context lengths, weight formats and options of this repository's own
workloads (the tiny, 1B- and 8B-shaped decoders; fp32, bf16, FP8 and int4 weights; normalised query / key heads);
`draw` gives more cases of the same ranges.

A case fixes every size, so that its bytes and operations can be counted; weights, tokens, block tables, logits and random
numbers come from the seed.  The caches that decode steps and chunks read are filled by the library's own prefill, as a
running node's are.  Model passes return the logits, whole: they depend on every key and value in the cache of their
sequence, the ones written by the pass among them (the pool itself is opaque to a caller).  The greedy tokens are asked
for as well, as a serving loop does, but not returned: they are the argmax of the returned logits, and on random-init
weights a near-tie falls either way with the last bits of a logit.
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

from paper_2603_20661_amd import binding as B
from paper_2603_20661_amd import synth

_FORMATS = {"": synth.WDTYPE_BF16, "fp8wo": synth.WDTYPE_FP8WO, "int4wo128": synth.WDTYPE_INT4WO_128, "int4wo32": synth.WDTYPE_INT4WO_32}


def listed():
    return [
        # one decode step of the smallest model, four chats: nothing but launches and latency
        {"name": "decode-tiny-b4", "kind": "decode", "model": "tiny", "batch": 4, "lens": "uniform", "lo": 128, "hi": 144, "recipe": 0},
        # a single user's conversation on an otherwise idle node
        {"name": "decode-8b-b1", "kind": "decode", "model": "8b", "batch": 1, "lens": "uniform", "lo": 1041, "hi": 1041, "recipe": 0},
        # a small model under an ordinary load: the 1B-shaped workload half-way through its generation
        {"name": "decode-1b-b32", "kind": "decode", "model": "1b", "batch": 32, "lens": "uniform", "lo": 576, "hi": 2112, "recipe": 1},
        # the ordinary load of a node: the 8B-shaped workload half-way through its generation
        {"name": "decode-8b-b64", "kind": "decode", "model": "8b", "batch": 64, "lens": "lognormal", "lo": 144, "hi": 4224, "recipe": 2},
        # a full node: many sequences, a few of them with long contexts
        {"name": "decode-8b-b128-zipf", "kind": "decode", "model": "8b", "batch": 128, "lens": "zipf", "lo": 256, "hi": 8192, "recipe": 2},
        # the two weight-only formats at the small batches they are chosen for
        {"name": "decode-8b-fp8wo-b16", "kind": "decode", "model": "8b-fp8wo", "batch": 16, "lens": "lognormal", "lo": 144, "hi": 4224, "recipe": 5},
        {"name": "decode-8b-int4wo128-b5", "kind": "decode", "model": "8b-int4wo128", "batch": 5, "lens": "lognormal", "lo": 144, "hi": 4224, "recipe": 6},
        # one short prompt arrives on an idle node: time to first token
        {"name": "prefill-8b-333", "kind": "prefill", "model": "8b", "batch": 1, "q": "uniform", "q_lo": 333, "q_hi": 333, "prefix": "none", "lo": 0, "hi": 0, "recipe": 0},
        # a call of the chunked schedule: 16 chunks of 512 tokens over cached prefixes of many lengths
        {"name": "prefill-8b-chunks-8192", "kind": "prefill", "model": "8b", "batch": 16, "q": "uniform", "q_lo": 512, "q_hi": 512, "prefix": "zipf", "lo": 256, "hi": 4096, "recipe": 2},
        # all prompts of the 1B-shaped workload, on the model with normalised query and key heads
        {"name": "prefill-1b-qknorm-b32", "kind": "prefill", "model": "1b-qknorm", "batch": 32, "q": "uniform", "q_lo": 512, "q_hi": 2048, "prefix": "none", "lo": 0, "hi": 0, "recipe": 1},
        # all prompts of the 8B-shaped workload in one call: the largest
        {"name": "prefill-8b-b64", "kind": "prefill", "model": "8b", "batch": 64, "q": "lognormal", "q_lo": 16, "q_hi": 4096, "prefix": "none", "lo": 0, "hi": 0, "recipe": 2},
        # the sampled tokens of a decode step: temperature and top-p of the paper's generation parameters
        {"name": "sample-b64", "kind": "sample", "batch": 64, "vocab": 128256, "temperature": 0.7, "top_p": 0.95},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "sample"])
    if kind == "sample":
        return {"kind": "sample", "batch": _log_int(rng, 1, 64), "vocab": rng.choice([1024, 32000, 128256]),
                "temperature": round(rng.uniform(0.5, 1.0), 3), "top_p": round(rng.uniform(0.7, 0.99), 3)}
    model = rng.choice(["tiny", "1b", "1b", "1b-qknorm", "1b-fp8wo", "8b", "8b", "8b-fp8wo", "8b-int4wo128", "8b-int4wo32"])
    recipe = rng.randrange(1 << 16)
    if kind == "decode":
        batch = _log_int(rng, 1, 128)
        top = max(64, min(8192, 120_000 // batch))       # at most about 120 000 tokens of context in the batch
        hi = _log_int(rng, 64, top)
        return {"kind": "decode", "model": model, "batch": batch, "lens": rng.choice(["uniform", "lognormal", "zipf"]),
                "lo": max(2, hi // rng.choice([2, 4, 16])), "hi": hi, "recipe": recipe}
    batch = _log_int(rng, 1, 48)
    q_hi = _log_int(rng, 16, max(16, min(2048, 32_768 // batch)))
    prefix = rng.choice(["none", "none", "uniform", "zipf"])
    hi = 0 if prefix == "none" else _log_int(rng, 64, max(64, min(8192, 49_152 // batch)))
    return {"kind": "prefill", "model": model, "batch": batch, "q": rng.choice(["uniform", "lognormal"]), "q_lo": max(1, q_hi // rng.choice([1, 2, 8])),
            "q_hi": q_hi, "prefix": prefix, "lo": 0 if prefix == "none" else max(1, hi // 16), "hi": hi, "recipe": recipe}


# ----------------------------------------------------------------------------------------------- sizes of a case
def _lengths(kind, n, lo, hi, recipe):
    if kind == "none":
        return np.zeros(n, np.int64)
    if kind == "uniform":
        return synth.lengths_uniform(recipe, n, lo, hi).astype(np.int64)
    if kind == "lognormal":      # median at a quarter of the longest
        return synth.lengths_lognormal(recipe, n, hi / 4.0, 0.6, lo, hi).astype(np.int64)
    return synth.lengths_zipf(recipe, n, 1.2, lo, hi).astype(np.int64)


def _sizes(case):
    """(new tokens, length after the call) of every sequence"""
    n = case["batch"]
    if case["kind"] == "decode":
        return np.ones(n, np.int64), _lengths(case["lens"], n, case["lo"], case["hi"], case["recipe"])
    q = _lengths(case["q"], n, case["q_lo"], case["q_hi"], case["recipe"])
    return q, q + _lengths(case["prefix"], n, case["lo"], case["hi"], case["recipe"] + 1)


def _shape(model):
    base, _, variant = model.partition("-")
    shape = synth.SHAPES[base]
    if variant == "qknorm":
        return dataclasses.replace(shape, qk_norm=1)
    return dataclasses.replace(shape, weight_dtype=_FORMATS[variant]) if variant else shape


# ------------------------------------------------------------------------------------------------------- inputs
_STREAM = None


def _stream():
    """The one stream of a program that drives one GPU (a decode step is captured, which the default stream does not allow)."""
    global _STREAM
    if _STREAM is None:
        _STREAM = torch.cuda.Stream()
    return _STREAM


def _make_blob(shape, gen, dev):
    """Random-init weights N(0, 0.02^2) in the blob format of include/www.h, made on the GPU; gains of 1."""
    entries, total = synth.blob_layout(shape)
    blob = torch.zeros(total, dtype=torch.uint8, device=dev)
    scale_at = {name: off for name, off, *_ in entries if name.endswith(".scale")}
    for name, off, rows, cols, dt in entries:
        n = rows * cols
        if name.endswith(".scale"):
            continue
        if name.endswith("norm"):
            blob[off:off + 4 * n].view(torch.float32).fill_(1.0)
        elif dt == synth.WDTYPE_F32:
            blob[off:off + 4 * n].view(torch.float32).normal_(0.0, 0.02, generator=gen)
        elif dt == synth.WDTYPE_BF16:
            blob[off:off + 2 * n].view(torch.bfloat16).normal_(0.0, 0.02, generator=gen)
        else:
            w = torch.empty(n, dtype=torch.float32, device=dev).normal_(0.0, 0.02, generator=gen)
            at = scale_at[name + ".scale"]
            if dt == synth.WDTYPE_FP8WO:
                scale = w.abs().max() / 448.0
                blob[at:at + 4].view(torch.float32).copy_(scale.view(1))
                blob[off:off + n].copy_((w / scale).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8))
            else:
                group = synth.INT4_GROUP[dt]
                g = w.view(-1, group)
                scale = (g.abs().amax(dim=1, keepdim=True) / 7.0).to(torch.bfloat16)
                blob[at:at + 2 * scale.numel()].view(torch.bfloat16).copy_(scale.view(-1))
                c = (g / scale.float()).round_().add_(8.0).clamp_(0.0, 15.0).to(torch.uint8).view(-1, 2)
                blob[off:off + n // 2].copy_(c[:, 0] | (c[:, 1] << 4))
            del w
    return blob


def _prepare_model(case, seed):
    dev = torch.device("cuda:0")
    shape = _shape(case["model"])
    gen = torch.Generator(device=dev).manual_seed(seed)
    q, seq = _sizes(case)
    n, prefix = len(q), seq - q
    mbs = int((seq.max() + synth.KV_BLOCK) // synth.KV_BLOCK) + 1
    need = [int(s) // synth.KV_BLOCK + 1 for s in seq]
    num_blocks = sum(need) + 16
    fill_tokens = min(int(prefix.sum()), max(16384, int(prefix.max())))
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).to(dev)
    with torch.cuda.stream(_stream()):
        blob = _make_blob(shape, gen, dev)
        cfg = B.make_config(shape, n, mbs, max(int(q.sum()), fill_tokens, 1), num_blocks)
        model = B.Model(cfg, blob, stream=_stream())
        del blob
        # block tables scattered over the pool
        ids = torch.randperm(num_blocks, generator=gen, device=dev).to(torch.int32)
        table = torch.zeros((n, mbs), dtype=torch.int32, device=dev)
        at = 0
        for b, k in enumerate(need):
            table[b, :k] = ids[at:at + k]
            at += k
        draw_tokens = lambda count: torch.randint(0, shape.vocab, (count,), dtype=torch.int32, device=dev, generator=gen)
        # the cached context of every sequence, as many sequences a call as the workspace takes
        b0 = 0
        while b0 < n:
            b1, total = b0, 0
            while b1 < n and total + int(prefix[b1]) <= fill_tokens:
                total += int(prefix[b1])
                b1 += 1
            rows = [b for b in range(b0, b1) if prefix[b] > 0]
            if rows:
                p = i32(prefix[rows])
                B.www_prefill(model, draw_tokens(total), p, p, table[rows].contiguous(), stream=_stream())
            b0 = b1
        state = {"kind": case["kind"], "model": model, "tokens": draw_tokens(int(q.sum())), "q": i32(q), "seq": i32(seq), "table": table,
                 "logits": torch.empty((n, shape.vocab), dtype=torch.float32, device=dev),
                 "next": torch.empty(n, dtype=torch.int32, device=dev)}
    _stream().synchronize()
    return state


def _prepare_sample(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(seed)
    n, V = case["batch"], case["vocab"]
    with torch.cuda.stream(_stream()):
        # next-token logits as a language model has them: a few likely tokens and a long tail, falling with the logarithm of
        # the rank, more or less steeply from row to row; tokens in random order
        steep = 1.8 + 1.2 * torch.rand((n, 1), generator=gen, device=dev)
        logits = torch.empty((n, V), dtype=torch.float32, device=dev)
        for b in range(n):
            rank = torch.randperm(V, generator=gen, device=dev).add_(1).to(torch.float32)
            logits[b] = 12.0 - steep[b] * rank.log_()
        logits.add_(torch.randn((n, V), generator=gen, device=dev), alpha=0.2)
        state = {"kind": "sample", "logits": logits, "u": torch.rand(n, generator=gen, device=dev), "scratch": torch.empty_like(logits),
                 "out": torch.empty(n, dtype=torch.int32, device=dev), "temperature": case["temperature"], "top_p": case["top_p"]}
    _stream().synchronize()
    return state


def prepare(case, seed):
    return _prepare_sample(case, seed) if case["kind"] == "sample" else _prepare_model(case, seed)


def run(state):
    st = _stream()
    if state["kind"] == "sample":
        B.www_sample_top_p(state["logits"], state["temperature"], state["top_p"], state["u"], state["scratch"], state["out"], stream=st)
        return state["out"]
    if state["kind"] == "decode":
        B.www_decode_step(state["model"], state["tokens"], state["seq"], state["table"], state["logits"], state["next"], stream=st)
    else:
        B.www_prefill(state["model"], state["tokens"], state["q"], state["seq"], state["table"], state["logits"], state["next"], stream=st)
    return state["logits"]


# ------------------------------------------------------------------------------------------------- work and bounds
def work(case):
    if case["kind"] == "sample":
        n = case["batch"] * case["vocab"]
        return {"bytes": 4.0 * n + 8.0 * case["batch"], "flops": 6.0 * n}     # each logit: scaled, its exponential, one sum
    s = _shape(case["model"])
    q, seq = (a.astype(np.float64) for a in _sizes(case))
    n, T, prefix = len(q), float(q.sum()), seq - q
    QD, KD, hd, L = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim, s.head_dim, s.n_layers
    per_layer = (QD + 2 * KD) * s.d_model + s.d_model * QD + 3 * s.ffn_dim * s.d_model   # weights
    per_weight = {synth.WDTYPE_F32: 4.0, synth.WDTYPE_BF16: 2.0, synth.WDTYPE_FP8WO: 1.0, synth.WDTYPE_INT4WO_128: 0.5 + 2 / 128,
                  synth.WDTYPE_INT4WO_32: 0.5 + 2 / 32}[s.weight_dtype]
    embed = 4.0 if s.weight_dtype == synth.WDTYPE_F32 else 2.0
    kv_token = L * 2 * s.n_kv_heads * (hd * 2 + 4)       # 16-bit codes and one scale per vector, all layers
    head = s.vocab * s.d_model
    moved = (L * per_layer + head) * per_weight + T * s.d_model * embed + n * s.vocab * 4.0
    moved += float(prefix.sum()) * kv_token + T * kv_token                               # cached context read, new entries written
    # every new token runs through all layers, except that the last layer's attention, output, gate / up and down products
    # are needed at a sequence's last token only, and the output head there as well; a query meets prefix + its own place
    last_layer_only = per_layer - (QD + 2 * KD) * s.d_model
    pairs = float(np.sum(q * prefix + q * (q + 1) / 2))
    flops = 2.0 * (T * (L * per_layer - last_layer_only) + n * (last_layer_only + head))
    flops += 4.0 * QD * (pairs * (L - 1) + float(seq.sum()))
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    if case["kind"] == "sample":
        return {"differ": 0.01}      # a draw that lies within fp32 rounding of a boundary may take the neighbouring token
    # Measured: a prompt through the prefill path (16-bit operands) against the same prompt token by token through the decode
    # path (operands of twice the bits): rel 2.0e-3 and max 9.7e-3 on the 8B shape, 4.3e-4 and 1.9e-3 on the two small ones.
    return {"rel": 8e-3, "max": 4e-2} if case["model"].startswith("8b") else {"rel": 2e-3, "max": 1e-2}
