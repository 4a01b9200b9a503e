"""The masked attention calls whose speed is tracked: sizes, inputs, one pass, and its compulsory work.

A pass is one forward through the public entry points (`Plan.forward`) on a plan that was built, and
prepared for the call shape, beforehand; the one exception is the kind "fresh", where every pass
brings a new dense mask and pays for its analysis.  Masks are static per model, so a case fixes its
mask (the mask's own seed is part of the case) and the seed given to `prepare` draws Q, K and V.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2506_06095_amd as smha
import workloads as W

_TORCH = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}


def _case(kind, B, H, S, d, dtype="f16", **kw):
    return dict(kind=kind, B=B, H=H, S=S, Sk=kw.pop("Sk", S), d=d, dtype=dtype, out=kw.pop("out", dtype),
                layout=kw.pop("layout", "bhsd"), std=kw.pop("std", 1.0), mask_seed=kw.pop("mask_seed", 1), **kw)


def listed():
    cases = [
        # smallest call: one short window-attention sentence with two heads; launch latency is the whole of it
        _case("window", 1, 2, 128, 64, band=16, name="tiny_window"),
        # encoder batch with Longformer attention at BERT-Base head sizes (window 64 either side, 8 global tokens)
        _case("longformer", 8, 12, 512, 64, band=64, n_global=8, name="longformer_bert"),
        # autoregressive model with strided sparse attention (local band plus every 128th key)
        _case("strided", 4, 16, 2048, 64, band=127, stride=128, name="strided_causal"),
        # learned block-sparse attention, another mask for every head
        _case("blocks", 2, 16, 4096, 64, "bf16", block=64, fill=0.10, mask_seed=4, name="random_blocks_bf16"),
        # the headline workload: one long document, BigBird blocks, padded to 8192
        _case("bigbird_blocks", 1, 32, 8192, 128, block=64, fill=0.0, std=0.5, mask_seed=5, max_pad=1023,
              name="bigbird_8k"),
        # prefill of a decoder: dense causal, a full batch of long sequences (the largest call)
        _case("causal", 16, 12, 4096, 128, name="causal_large"),
        # the same direction at a smaller model's head size, bfloat16, a sequence that fills no tile
        _case("causal", 4, 16, 2047, 64, "bf16", name="causal_ragged_bf16"),
        # BigBird as token classifiers use it: window, global tokens and 10 % random 32 x 32 blocks
        _case("bigbird", 16, 12, 2048, 64, band=32, n_global=32, block=32, fill=0.10, mask_seed=1024,
              name="bigbird_bert"),
        # padded batch straight from a projection ([batch, seq, head, dim] in memory), a head size between the
        # kernels' widths, full-precision output for a following fp32 normalisation
        _case("window", 4, 12, 3001, 80, "bf16", band=64, out="f32", layout="bshd", max_pad=700, name="window_padded"),
        # scattered keys (hash buckets, retrieved tokens): the per-row format's ground
        _case("scattered", 4, 16, 2048, 64, per_row=8, name="scattered_rows"),
        # a chunk of queries against a long cache (chunked prefill: band of 1024 and 64 sink keys)
        _case("chunk", 2, 16, 2048, 128, Sk=16384, band=1023, n_global=64, name="chunk_of_16k"),
        # a mask that is new with every input (document structure): analysis and forward in one pass
        _case("fresh", 1, 12, 1024, 64, band=32, n_global=32, name="fresh_mask"),
    ]
    return cases


def _loguniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A length in [lo, hi], log-uniform; half of them a multiple of 64, the rest as they fall."""
    n = _loguniform(rng, lo, hi)
    return max(lo, n // 64 * 64) if rng.random() < 0.5 else n


def draw(rng):
    largest = work(_largest())
    while True:
        kind = rng.choice(["window", "window", "longformer", "longformer", "causal", "causal", "bigbird", "bigbird",
                           "bigbird_blocks", "bigbird_blocks", "blocks", "blocks", "strided", "scattered", "chunk",
                           "fresh"])
        H = rng.choice([2, 4, 8, 12, 12, 16, 16, 20, 32])
        d = rng.choice([64, 64, 64, 128, 128, 128, 32, 80, 96, 112, 160, 256])
        dtype = rng.choice(["f16", "f16", "bf16"])
        kw = dict(out="f32" if rng.random() < 0.15 else dtype, layout="bshd" if rng.random() < 0.3 else "bhsd",
                  std=rng.choice([0.5, 1.0]), mask_seed=rng.randrange(1, 1 << 30))
        B, S = _loguniform(rng, 1, 16), _size(rng, 128, 4096)
        if kind in ("window", "longformer", "bigbird", "strided", "fresh"):
            kw["band"] = _loguniform(rng, 16, 512 if kind == "window" else 128)
        if kind in ("longformer", "bigbird", "fresh"):
            kw["n_global"] = _loguniform(rng, 1, 64)
        if kind == "bigbird":
            kw.update(block=32, fill=rng.uniform(0.03, 0.15))
        if kind == "blocks":
            kw.update(block=rng.choice([32, 64, 64, 128]), fill=rng.uniform(0.05, 0.25))
            B, S = _loguniform(rng, 1, 4), _size(rng, 512, 4096)
        if kind == "bigbird_blocks":
            kw.update(block=64, fill=0.0)
            B, S = _loguniform(rng, 1, 4), _size(rng, 1024, 8192)
        if kind == "strided":
            kw["stride"] = _loguniform(rng, 32, 256)
        if kind == "scattered":
            kw["per_row"] = _loguniform(rng, 2, 16)
            B, S = _loguniform(rng, 1, 8), _size(rng, 512, 4096)
        if kind == "chunk":
            kw.update(Sk=_size(rng, 4096, 16384), band=_loguniform(rng, 128, 2048), n_global=_loguniform(rng, 4, 64))
            B, S = _loguniform(rng, 1, 4), _size(rng, 64, 2048)
        if kind == "fresh":
            B, S = 1, _size(rng, 256, 2048)
        if kind in ("window", "longformer", "causal", "bigbird", "bigbird_blocks") and rng.random() < 0.3:
            kw["max_pad"] = S // 4
        case = _case(kind, B, H, S, d, dtype, **kw)
        w = work(case)
        if w["flops"] <= largest["flops"] and w["bytes"] <= largest["bytes"]:
            return case


def _largest():
    return next(c for c in listed() if c["name"] == "causal_large")


def _spec(case):
    """The mask's description, for the kinds that have one."""
    kind, f, kw = case["kind"], 0, {}
    if kind in ("window", "longformer", "bigbird"):
        f, kw = W.WINDOW, dict(window_left=case["band"], window_right=case["band"])
    if kind in ("longformer", "bigbird"):
        f, kw = f | W.GLOBAL, dict(kw, n_global=case["n_global"])
    if kind in ("bigbird", "blocks"):
        f, kw = f | W.BLOCK_RANDOM, dict(kw, block=case["block"], keep_p=case["fill"], per_head=kind == "blocks")
    if kind == "bigbird_blocks":
        f, kw = W.BIGBIRD, dict(block=case["block"], n_window_blocks=3, n_global_blocks=2, n_random_blocks=3)
    if kind == "causal":
        f = W.CAUSAL
    if kind == "strided":
        f, kw = W.CAUSAL | W.WINDOW | W.STRIDED, dict(window_left=case["band"], stride=case["stride"])
    if case.get("max_pad"):
        f |= W.PADDING
        kw["valid_len"] = tuple(case["S"] - W.mix64(W.mix64(case["mask_seed"]) ^ (0x70616421 + b)) % (case["max_pad"] + 1)
                                for b in range(case["B"]))
    return W.MaskSpec(flags=f, seed=case["mask_seed"], **kw)


def _dense_mask(case, seed, device):
    """uint8 [1, 1, S, Sk]: the masks that no description covers."""
    S, Sk = case["S"], case["Sk"]
    g = torch.Generator(device=device).manual_seed(seed)
    i = torch.arange(Sk - S, Sk, device=device)[:, None]  # the queries' positions: the last S of the sequence
    j = torch.arange(Sk, device=device)[None, :]
    if case["kind"] == "scattered":
        m = torch.zeros(S, Sk, dtype=torch.uint8, device=device)
        m.scatter_(1, torch.randint(Sk, (S, case["per_row"]), device=device, generator=g), 1)
        m.fill_diagonal_(1)
    elif case["kind"] == "chunk":
        m = (j <= i) & ((i - j <= case["band"]) | (j < case["n_global"]))
    else:  # "fresh": band and a number of global tokens at places of their own
        at = torch.zeros(Sk, dtype=torch.bool, device=device)
        at[torch.randperm(Sk, device=device, generator=g)[: case["n_global"]]] = True
        m = ((i - j).abs() <= case["band"]) | at[None, :]
    return m.to(torch.uint8)[None, None].contiguous()


def _tensor(case, rows, g):
    B, H, d = case["B"], case["H"], case["d"]
    shape = (B, rows, H, d) if case["layout"] == "bshd" else (B, H, rows, d)
    x = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(case["std"]).to(_TORCH[case["dtype"]])
    return x.transpose(1, 2) if case["layout"] == "bshd" else x


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    state = {"case": case, "q": _tensor(case, case["S"], g), "k": _tensor(case, case["Sk"], g),
             "v": _tensor(case, case["Sk"], g)}
    if case["kind"] == "fresh":
        state["mask"] = _dense_mask(case, seed, "cuda")
        return state
    if case["kind"] in ("scattered", "chunk"):
        make = smha.Plan.from_dense if case["S"] == case["Sk"] else smha.Plan.from_dense_rect
        plan = make(_dense_mask(case, case["mask_seed"], "cuda"), head_dim=case["d"])
    else:
        plan = smha.Plan.from_desc(_spec(case), case["B"], case["H"], case["S"], head_dim=case["d"])
    plan.prepare(case["B"], case["H"], case["d"])
    state["plan"] = plan
    return state


def run(state):
    case = state["case"]
    out = _TORCH[case["out"]]
    if case["kind"] == "fresh":
        with smha.Plan.from_dense(state["mask"], head_dim=case["d"]) as plan:
            return plan.forward(state["q"], state["k"], state["v"], out_dtype=out)
    return state["plan"].forward(state["q"], state["k"], state["v"], out_dtype=out)


def _entries(case):
    """Unmasked (query, key) pairs, summed over batch and heads."""
    B, H, S, Sk = case["B"], case["H"], case["S"], case["Sk"]
    if case["kind"] == "scattered":  # (expected number of different keys in a row)
        return B * H * S * Sk * (1 - (1 - 1 / Sk) ** (case["per_row"] + 1))
    if case["kind"] == "chunk":
        i = np.arange(Sk - S, Sk)
        return B * H * float((np.minimum(i, case["band"]) + 1 + np.clip(i - case["band"], 0, case["n_global"])).sum())
    if case["kind"] == "fresh":  # (band, plus the expected number of global keys outside it)
        i = np.arange(S)
        band = (np.minimum(i, case["band"]) + 1 + np.minimum(S - 1 - i, case["band"])).astype(float)
        return B * H * float((band + (S - band) * min(1.0, case["n_global"] / S)).sum())
    return _entries_of_spec(_spec(case), B, H, S)


@functools.lru_cache(maxsize=256)
def _entries_of_spec(spec, B, H, S):
    with smha.Plan.from_desc(spec, B, H, S, device_id=-2) as plan:  # (host analysis only)
        info = plan.info()
    return info["nnz"] * (B // info["Bm"]) * (H // info["Hm"])


def work(case):
    item, out = 2, torch.empty(0, dtype=_TORCH[case["out"]]).element_size()
    heads = case["B"] * case["H"] * case["d"]
    keys = case["Sk"]
    if case["kind"] == "chunk":  # (the keys that no query attends are not read)
        keys = min(keys, case["S"] + case["band"] + case["n_global"])
    nbytes = heads * (case["S"] * (item + out) + 2 * keys * item)
    if case["kind"] == "fresh":
        nbytes += case["S"] * case["Sk"]
    return {"bytes": int(nbytes), "flops": int(4 * case["d"] * _entries(case))}


def tolerance(case):
    """About four times the largest error against float64 on the same inputs (all listed and 14 drawn cases)."""
    if case["dtype"] == "f16":  # probabilities and output rounded to binary16: 2.0e-4 to 3.0e-4, largest difference 3.9e-3
        return {"rel": 1.2e-3, "max": 1.6e-2}
    if case["out"] == "f32":    # bfloat16 products, probabilities to 2^-17, fp32 sums: 4.1e-6 to 5.1e-6, largest 3.7e-5
        return {"rel": 2e-5, "max": 1.5e-4}
    return {"rel": 6.6e-3, "max": 1.6e-2}  # the output's rounding to bfloat16: 1.6e-3 to 1.7e-3, largest 3.9e-3
