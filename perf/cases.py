"""The work a user of the library has it do, as cases that can be timed and compared.

A case is one of four kinds of call through the public entry points of ``paper_2407_07304_amd.slimattn``:

  prefill   attention of a prompt, bf16 or INT8 K/V, bf16 or fp32 output
  cache     the same attention that also writes the prompt's INT8 K/V cache
  quantise  INT8 codes and scales of K (and V) that are already there
  decode    one step of token generation: the new token's K and V into the cache, then attention over the cache

K, V and Q are drawn i.i.d. N(0, 1) like the repository's own workloads (``inputs.py``), on the device.  ``listed()``
holds fixed sizes from the repository's configurations, tests and benchmark, ``draw()`` the ranges they stand for.
"""
import math

import torch

from paper_2407_07304_amd import slimattn as sa


def _prefill(name, batch, q_heads, kv_heads, seq_len, head_dim=128, causal=True, kv="bf16", out="bf16", kind="prefill"):
    return {"name": name, "kind": kind, "batch": batch, "q_heads": q_heads, "kv_heads": kv_heads, "seq_len": seq_len,
            "head_dim": head_dim, "causal": causal, "kv": kv, "out": out}


def _quantise(name, batch, kv_heads, seq_len, head_dim=128, pair=True):
    return {"name": name, "kind": "quantise", "batch": batch, "kv_heads": kv_heads, "seq_len": seq_len,
            "head_dim": head_dim, "pair": pair}


def _decode(name, batch, q_heads, kv_heads, kv_len, head_dim=128, entry="workspace"):
    return {"name": name, "kind": "decode", "batch": batch, "q_heads": q_heads, "kv_heads": kv_heads, "kv_len": kv_len,
            "head_dim": head_dim, "entry": entry}


def listed():
    return [
        # one user's chat turn, short cache, under graph-friendly calls: latency of the launches is all there is
        _decode("decode_one_user", 1, 32, 32, 1000, entry="static"),
        # one user with a long document, grouped heads: one sequence has to fill the whole chip
        _decode("decode_long_document", 1, 64, 8, 32768),
        # the benchmark's decode: 16 sequences, multi-head, 8192 cached tokens each
        _decode("decode_batch16_mha", 16, 32, 32, 8192),
        # the benchmark's grouped-query decode
        _decode("decode_batch16_gqa", 16, 64, 8, 8192),
        # a serving batch whose sequences have all got differently far (lengths spread over the allocated cache)
        _decode("decode_ragged_batch", 48, 32, 8, 3001, entry="varlen"),
        # the parity configuration: a short prompt, small heads, fp32 output
        _prefill("prefill_short_fp32", 1, 8, 8, 512, head_dim=64, out="f32"),
        # the headline configuration
        _prefill("prefill_2k", 1, 32, 32, 2048),
        # the same heads over an INT8 cache
        _prefill("prefill_4k_int8", 1, 32, 32, 4096, kv="int8"),
        # long-context grouped-query prefill over an INT8 cache: the largest
        _prefill("prefill_32k_gqa_int8", 1, 64, 8, 32768, kv="int8"),
        # a batch of prompts of an odd length, attended to and put into the cache in one call
        _prefill("prefill_batch_cache", 4, 32, 8, 777, kind="cache"),
        # the prompt's K and V into the cache after a prefill
        _quantise("quantise_2k_pair", 1, 32, 2048),
        # a whole batch's keys at once (the benchmark's cache)
        _quantise("quantise_stream", 16, 32, 8192, pair=False),
    ]


_HEADS = ((8, 8), (32, 32), (32, 8), (64, 8), (16, 2), (4, 4))
_MOST_FLOPS = 8.0e12          # of a drawn prefill: below the largest listed one
_MOST_CACHE = 500 << 20       # bytes of K codes of a drawn decode or quantiser call


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("prefill", "prefill", "cache", "quantise", "decode", "decode", "decode"))
    head_dim = rng.choice((64, 128, 128))
    q_heads, kv_heads = rng.choice(_HEADS)
    if kind in ("prefill", "cache"):
        causal = rng.random() < 0.85     # the rest: bidirectional attention
        while True:
            seq_len, batch = _log_int(rng, 48, 16384), _log_int(rng, 1, 16)
            c = _prefill("", batch, q_heads, kv_heads, seq_len, head_dim, causal,
                         "int8" if kind == "prefill" and rng.random() < 0.5 else "bf16",
                         "f32" if rng.random() < 0.2 else "bf16", kind)
            if work(c)["flops"] <= _MOST_FLOPS:
                break
    elif kind == "quantise":
        while True:
            seq_len, batch = _log_int(rng, 32, 32768), _log_int(rng, 1, 32)
            if batch * kv_heads * seq_len * head_dim <= _MOST_CACHE // 2:
                break
        c = _quantise("", batch, kv_heads, seq_len, head_dim, rng.random() < 0.7)
    else:
        while True:
            kv_len, batch = _log_int(rng, 64, 65536), _log_int(rng, 1, 128)
            if batch * kv_heads * kv_len * head_dim <= _MOST_CACHE:
                break
        entry = rng.choice(("workspace", "varlen", "static"))
        if entry == "static" and batch * q_heads > 256:   # (the library's own scratch is meant for small steps)
            entry = "workspace"
        c = _decode("", batch, q_heads, kv_heads, kv_len, head_dim, entry)
    del c["name"]
    return c


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=dev, dtype=torch.bfloat16)

    b, hkv, d = case["batch"], case["kv_heads"], case["head_dim"]
    st = {"case": dict(case), "scale": 1.0 / math.sqrt(d)}
    if case["kind"] in ("prefill", "cache"):
        s = case["seq_len"]
        st["q"], st["k"], st["v"] = normal(b, case["q_heads"], s, d), normal(b, hkv, s, d), normal(b, hkv, s, d)
        st["k_scale"] = st["v_scale"] = None
        if case["kv"] == "int8":
            st["k"], st["k_scale"], st["v"], st["v_scale"] = sa.kv_quant_int8_pair(st["k"], st["v"])
        st["out_dtype"] = torch.float32 if case["out"] == "f32" else torch.bfloat16
    elif case["kind"] == "quantise":
        st["k"] = normal(b, hkv, case["seq_len"], d)
        if case["pair"]:
            st["v"] = normal(b, hkv, case["seq_len"], d)
    else:
        t, hq = case["kv_len"], case["q_heads"]
        st["kc"], st["ks"] = sa.kv_quant_int8(normal(b, hkv, t, d))
        st["vc"], st["vs"] = sa.kv_quant_int8(normal(b, hkv, t, d))
        st["q"], st["k_new"], st["v_new"] = normal(b, hq, 1, d), normal(b, hkv, 1, d), normal(b, hkv, 1, d)
        if case["entry"] == "varlen":   # each sequence has got somewhere between an eighth of the cache and all of it
            lens = torch.randint(max(1, t // 8), t + 1, (b,), generator=gen, device=dev, dtype=torch.int32)
        else:
            lens = torch.full((b,), t, device=dev, dtype=torch.int32)
        st["lens"], st["positions"] = lens, lens - 1
        # what a serving loop keeps from step to step
        st["out"] = torch.empty((b, hq, 1, d), dtype=torch.bfloat16, device=dev)
        if case["entry"] != "static":
            st["workspace"] = torch.empty(max(16, sa.slim_attn_decode_int8_workspace_bytes(b, hq, hkv, t, d)),
                                          dtype=torch.uint8, device=dev)
    return st


def run(state):
    c = state["case"]
    if c["kind"] == "prefill":
        return sa.slim_attn_prefill(state["q"], state["k"], state["v"], state["scale"], c["causal"], k_scale=state["k_scale"],
                                    v_scale=state["v_scale"], out_dtype=state["out_dtype"])
    if c["kind"] == "cache":
        return sa.slim_attn_prefill_emit_int8(state["q"], state["k"], state["v"], state["scale"], c["causal"],
                                              out_dtype=state["out_dtype"])
    if c["kind"] == "quantise":
        if c["pair"]:
            return sa.kv_quant_int8_pair(state["k"], state["v"])
        return sa.kv_quant_int8(state["k"])
    kc, ks, vc, vs = state["kc"], state["ks"], state["vc"], state["vs"]
    sa.kv_quant_int8_append(state["k_new"], kc, ks, state["positions"])
    sa.kv_quant_int8_append(state["v_new"], vc, vs, state["positions"])
    if c["entry"] == "static":
        out = sa.slim_attn_decode_int8_static(state["q"], kc, ks, vc, vs, state["scale"], state["out"])
    elif c["entry"] == "varlen":
        out = sa.slim_attn_decode_int8_varlen(state["q"], kc, ks, vc, vs, state["lens"], state["scale"], out=state["out"],
                                              workspace=state["workspace"])
    else:
        out = sa.slim_attn_decode_int8(state["q"], kc, ks, vc, vs, state["scale"], out=state["out"],
                                       workspace=state["workspace"])
    return {"out": out, "k_codes": kc, "k_scale": ks, "v_codes": vc, "v_scale": vs}


def work(case):
    b, hkv, d = case["batch"], case["kv_heads"], case["head_dim"]
    if case["kind"] in ("prefill", "cache"):
        s, hq = case["seq_len"], case["q_heads"]
        pairs = s * (s + 1) // 2 if case["causal"] else s * s
        q_bytes, out_bytes = 2 * b * hq * s * d, (4 if case["out"] == "f32" else 2) * b * hq * s * d
        codes = 2 * b * hkv * s * (d + 4)    # K and V codes with their scales
        kv_bytes = codes if case["kv"] == "int8" else 4 * b * hkv * s * d
        written = codes if case["kind"] == "cache" else 0
        return {"bytes": q_bytes + kv_bytes + out_bytes + written, "flops": 4 * b * hq * d * pairs}
    if case["kind"] == "quantise":
        n = b * hkv * case["seq_len"] * (2 if case["pair"] else 1)
        return {"bytes": n * (3 * d + 4), "flops": 3 * n * d}
    t, hq = case["kv_len"], case["q_heads"]
    if case["entry"] == "varlen":
        t = (t + max(1, t // 8)) / 2         # the mean of the lengths that prepare() draws
    return {"bytes": 2 * b * hkv * t * (d + 4) + 4 * b * hq * d + 2 * b * hkv * (3 * d + 4), "flops": 4 * b * hq * t * d}


def tolerance(case):
    # codes and scales are defined bit for bit; the attention rounds its probabilities and its results to bf16
    # (the fp32 output as well: its probabilities are bf16 operands of the second product)
    if case["kind"] == "quantise":
        return "exact"
    return {"rel": 1e-2, "differ": 0.0}
