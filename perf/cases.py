"""The work a user of this library has it do, as cases that can be timed and compared.

A case is one layer (or a few) of a served model's KV cache, driven through the Python binding:
  step      one decode step: append one token per sequence and attend over the whole cache
            (RkvCache.decode_step), for `layers` layers one after the other;
  verify    a multi-token step: `queries` tokens are appended, read the cache together with the causal
            mask, and the rejected ones are rolled back (speculative decoding);
  prefill   prompts arrive: the caches are reset, the sink tokens are identified from the activations,
            and all tokens are compressed and appended (RkvCache.quantize_append / _ragged).
Keys carry a few strong channels per head, the first tokens of a sequence are sinks (massive
activations in the block's output, keys that draw attention), values and queries are plain noise:
the structure of real keys and values.  Shapes are
those of the benchmark's configurations (32 or 40 heads of 128, 8 KV heads under 32 query heads,
contexts from 512 to 32768), and generic ones in between.
"""
import math

import torch

import paper_2501_16383_amd as R

D = 128
SLACK = 64          # decode steps before a cache is full and its slots go to the next request of the same prompt

_BASE = dict(kind="step", batch=1, q_heads=32, kv_heads=32, context=4096, layers=1, rot_heads=4, sinks=4, theta=10000.0, bits=2,
             quant_group=128, span=128, meta=0, shortest=0, queries=1)


def _case(**kw):
    c = dict(_BASE)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call there is in use: one sequence, half a thousand tokens, one layer (latency and launches)
        _case(name="step_tiny", context=512, rot_heads=2, sinks=1),
        # one user chatting: a few layers of one sequence, every kernel far from filling the chip
        _case(name="step_single", context=4096, layers=4),
        # the headline configuration: 40 heads, batch 16, 4096 tokens
        _case(name="step_batch", batch=16, q_heads=40, kv_heads=40),
        # grouped-query serving: 32 query heads on 8 KV heads, batch 32, 8192 tokens
        _case(name="step_gqa", batch=32, kv_heads=8, context=8192, theta=500000.0),
        # one long document
        _case(name="step_long", context=32768),
        # continuous batching: sequences of different, odd lengths
        _case(name="step_ragged", batch=8, context=4090, shortest=1021),
        # speculative decoding: four drafted tokens verified at once
        _case(name="verify_gqa", kind="verify", batch=8, kv_heads=8, theta=500000.0, queries=4),
        # wider codes where quality matters more than memory
        _case(name="step_4bit", batch=8, bits=4),
        # small quantization groups with 8-bit metadata
        _case(name="step_group32", batch=8, quant_group=32, meta=1),
        # the reorder over the whole token row, as the calibration algorithm is printed
        _case(name="step_whole_row", batch=8, span=4096),
        # a batch of prompts of one length
        _case(name="prefill", kind="prefill", batch=4, q_heads=40, kv_heads=40),
        # prompts of different, odd lengths under grouped-query heads
        _case(name="prefill_ragged", kind="prefill", batch=8, kv_heads=8, context=1531, shortest=37, theta=500000.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 7 + ["verify"] * 2 + ["prefill"] * 2)
    kv = rng.choice([4, 8, 8, 16, 32, 40])
    rep = rng.choice([1, 1, 2, 3, 4, 4, 7, 8]) if kv <= 16 else 1
    c = _case(kind=kind, q_heads=kv * rep, kv_heads=kv, rot_heads=rng.choice([2, 4, 4, 4]), sinks=rng.choice([0, 1, 4, 4]),
              theta=500000.0 if rep > 1 else 10000.0, meta=rng.choice([0, 0, 1]))
    if kind == "prefill":
        c["context"] = _log_int(rng, 17, 4096)
        c["batch"] = max(1, min(_log_int(rng, 1, 32), 16384 * 40 // (kv * c["context"])))
        if c["batch"] > 1 and rng.random() < 0.5:
            c["shortest"] = max(1, int(c["context"] * rng.uniform(0.02, 0.9)))
        c["bits"] = rng.choice([2, 2, 2, 3, 4])
        return c
    c["context"] = _log_int(rng, 130, 32768)
    c["batch"] = _log_int(rng, 1, 32)
    most = 2_000_000                                         # cached (token, KV head) pairs
    if kind == "verify":
        c["queries"] = rng.randint(2, 8)
        most = 2_000_000 // (rep * c["queries"])
    else:
        variant = rng.choice(["plain"] * 5 + ["bits", "group", "span"])
        if variant == "bits":
            c["bits"] = rng.choice([3, 4])
        elif variant == "group":
            c["quant_group"] = rng.choice([32, 64])
        elif variant == "span":
            c["span"] = rng.choice([c["rot_heads"], kv]) * D
        if variant != "plain":
            most = 1_000_000 // rep
        if rep == 1 and rng.random() < 0.2:
            c["layers"] = rng.choice([2, 4])
            most //= c["layers"]
    c["batch"] = max(1, min(c["batch"], most // (kv * c["context"])))
    c["context"] = min(c["context"], max(130, most // kv))
    if kind == "step" and c["span"] == D and c["batch"] > 1 and rng.random() < 0.3:
        c["shortest"] = max(1, int(c["context"] * rng.uniform(0.1, 0.9)))
    return c


def _slack(c):
    """Tokens between a prompt and a full cache."""
    return 0 if c["kind"] == "prefill" else min(SLACK, c["context"] // 4)


def _lengths(c):
    """Prompt lengths: all equal, or spread from `shortest` to the full context over the batch."""
    B, T = c["batch"], c["context"] - _slack(c)
    lo = min(c["shortest"] or T, T)
    return [int(round(lo + (T - lo) * b / max(B - 1, 1))) if B > 1 else T for b in range(B)]


def _bytes_per_token(c):
    E = c["kv_heads"] * D
    return 2 * (E * c["bits"] // 8) + 2 * (E // c["quant_group"]) * (2 if c["meta"] else 4)


def _config(c):
    return R.RkvConfig(batch=c["batch"], n_q_heads=c["q_heads"], n_kv_heads=c["kv_heads"], max_tokens=c["context"],
                       max_sinks=c["sinks"], rot_heads=c["rot_heads"], quant_group=c["quant_group"], bits=c["bits"],
                       perm_span=c["span"], rope_theta=c["theta"], meta_format=c["meta"])


def _gains(c, g, dev):
    """Magnitude of every key channel: six strong channels (10 to 50 times the rest) in each head."""
    gain = torch.ones(c["kv_heads"], D, device=dev)
    where = torch.rand(c["kv_heads"], D, generator=g, device=dev).argsort(1)[:, :6]
    return gain.scatter_(1, where, torch.rand(c["kv_heads"], 6, generator=g, device=dev) * 40 + 10).half()


def _rows(c, g, gain, batch, n, dev):
    shape = (batch, n, c["kv_heads"], D)
    k = torch.randn(shape, generator=g, device=dev, dtype=torch.float16).mul_(gain)
    v = torch.randn(shape, generator=g, device=dev, dtype=torch.float16)
    return k, v


def prepare(case, seed):
    c, dev = case, torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    cfg, lens = _config(c), _lengths(c)
    B, n, ragged = c["batch"], max(lens), len(set(lens)) > 1
    s = dict(case=c, lens=lens, ragged=ragged, caches=[], k=[], v=[], q=[], out=[])
    mask = None
    if c["sinks"] and c["kind"] != "prefill":
        mask = torch.zeros(B, n, dtype=torch.uint8, device=dev)
        mask[:, :c["sinks"]] = 1
    scratch = torch.empty(R.query_sizes(cfg)[1], dtype=torch.uint8, device=dev)
    for _ in range(c["layers"]):
        gain = _gains(c, g, dev)
        cache = R.RkvCache(cfg, device=dev, scratch=scratch)
        cache.set_perm(R.calibrate_perm(cfg, _rows(c, g, gain, 1, 256, dev)[0][0]))
        k, v = _rows(c, g, gain, B, n, dev)
        k[:, :c["sinks"]] *= 2                               # sinks draw attention, but leave some to the other tokens
        v[:, :c["sinks"]] *= 2
        if c["kind"] == "prefill":
            s["k"].append(k)
            s["v"].append(v)
        else:
            if ragged:
                cache.quantize_append_ragged(k, v, lens, mask)
            else:
                cache.quantize_append(k, v, mask)
            del k, v
            nq = c["queries"]
            k, v = _rows(c, g, gain, B, nq, dev)
            s["k"].append(k)
            s["v"].append(v)
            q = torch.randn(B, nq, c["q_heads"], D, generator=g, device=dev, dtype=torch.float16)
            s["q"].append(q if c["kind"] == "verify" else q[:, 0].contiguous())
            s["out"].append(torch.empty(B, c["q_heads"], D, dtype=torch.float32, device=dev))
        s["caches"].append(cache)
    if c["kind"] == "verify":
        s["ahead"] = torch.arange(c["queries"], dtype=torch.int32, device=dev).repeat(B, 1)
    if c["kind"] == "prefill" and c["sinks"]:
        # the previous block's output, in which the sinks show as massive activations
        x = torch.randn(B, n, c["q_heads"] * D, generator=g, device=dev, dtype=torch.float16)
        where = torch.rand(B, min(lens), generator=g, device=dev).argsort(1)[:, :c["sinks"]]
        x[torch.arange(B, device=dev)[:, None], where, 77] = 500.0
        s["x"] = x
    return s


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "prefill":
        mask = R.select_sinks(s["x"], min(c["sinks"], s["x"].shape[1]))[1] if c["sinks"] else None
        for cache, k, v in zip(s["caches"], s["k"], s["v"]):
            cache.reset()
            if s["ragged"]:
                cache.quantize_append_ragged(k, v, s["lens"], mask)
            else:
                cache.quantize_append(k, v, mask)
        return [cache.mem for cache in s["caches"]] + ([mask] if mask is not None else [])
    if s["caches"][0].length + c["queries"] > c["context"]:  # full: the next request of the same prompt
        for cache in s["caches"]:
            cache.truncate(s["lens"])
    if c["kind"] == "verify":
        outs = []
        for cache, k, v, q in zip(s["caches"], s["k"], s["v"], s["q"]):
            at = cache.length
            pos = s["ahead"] + at
            cache.quantize_append(k, v)
            outs.append(cache.decode_attention_multi(q, pos))
            cache.truncate(at + (c["queries"] + 1) // 2)     # half of the drafted tokens are accepted
        return outs
    for cache, k, v, q, out in zip(s["caches"], s["k"], s["v"], s["q"], s["out"]):
        cache.decode_step(k, v, q, out=out)
    return s["out"]


def work(case):
    c = case
    E, n = c["kv_heads"] * D, c["rot_heads"] * D
    tokens = sum(_lengths(c)) + (0 if c["kind"] == "prefill" else c["batch"] * _slack(c) // 2)
    stored = tokens * _bytes_per_token(c)
    if c["kind"] == "prefill":
        act = c["batch"] * max(_lengths(c)) * c["q_heads"] * D * 2 if c["sinks"] else 0
        # rotation (one addition per butterfly stage) of the keys, then the extremes, a division and a rounding for keys and values
        return {"bytes": c["layers"] * (tokens * 4 * E + stored) + act, "flops": c["layers"] * tokens * E * (math.log2(n) + 8)}
    new = c["batch"] * c["queries"]
    bytes_ = stored + new * (4 * E + _bytes_per_token(c)) + new * c["q_heads"] * D * (2 + 4)
    # per cached element: dequantization of K and V, rotation and RoPE of K; per query: q.k and p.v
    flops = tokens * E * (4 + math.log2(n) + 3) + 4 * tokens * c["queries"] * c["q_heads"] * D
    return {"bytes": c["layers"] * bytes_, "flops": c["layers"] * flops}


def tolerance(case):
    # Attention outputs against the same attention in float64 on the dequantized cache, over these cases and
    # drawn ones: at most 3.7e-6 of the norm, and 5.7e-5 in the largest single difference.  Cache bytes:
    # a code may fall on the other side of a rounding tie.
    return {"rel": 1.5e-5, "max": 2.3e-4, "differ": 1e-4}
