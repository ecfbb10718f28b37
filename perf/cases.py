"""The work that users of the fold step have it do, as measurable cases.

A case is one pass of a user's program: `steps` consecutive chunks of `n` tokens, each through `layers` layers, onto
caches that already hold `prev` tokens.  The pass rewinds the caches to `prev` rows (host-side bookkeeping) and calls
`KvFoldCache.step`, the package's public entry point, once per chunk and layer.  Outputs are everything a step
produces: the attention output, the log-sum-exp where it is asked for, and the K/V rows that joined the caches.

Keys of a case: dtype ("bf16" or "f32"), hq / hkv / d (query heads, KV heads, head dim), n, steps, layers, prev,
mode ("plain", "rope": rotary embedding inside the step, "window": sink + sliding-window mask, "noalloc": the step for
callers that cannot allocate), bits (0, or the 8 / 4 of the storage round trip), sink and window (the mask), lse.
"""
from __future__ import annotations

import math

import torch

from paper_2605_12471_amd import KvFoldCache
from paper_2605_12471_amd import inputs as I


def _case(name, dtype="bf16", hq=32, hkv=8, d=128, n=1, steps=1, layers=1, prev=0, mode="plain", bits=0, sink=0,
          window=0, lse=False):
    case = {"name": name, "dtype": dtype, "hq": hq, "hkv": hkv, "d": d, "n": n, "steps": steps, "layers": layers,
            "prev": prev, "mode": mode, "bits": bits, "sink": sink, "window": window, "lse": lse}
    if name is None:
        del case["name"]
    return case


def listed():
    return [
        # The smallest fold of the benchmark definition: four chunks of 128 tokens, one layer, fp32 (the precision
        # reference of a small model's layer); nothing but launches, latency and host time.
        _case("tiny_fold_f32", dtype="f32", hq=4, hkv=1, d=64, n=128, steps=4),
        # Greedy decoding after a short document: one token through 16 layers of Llama-3.1-8B shape, each with its own
        # 4 K-token cache of a length that is no multiple of anything.
        _case("decode_4k_16_layers", n=1, layers=16, prev=4187),
        # Greedy decoding after the long chain: one token against a 128K-token cache, bound by reading the cache.
        _case("decode_128k", n=1, prev=130941, lse=True),
        # The question that follows the document in the needle protocol has a length of its own: 37 tokens, rotary
        # embedding inside the step, on a 32K-token cache, two layers.
        _case("question_rope_32k", n=37, layers=2, prev=32768, mode="rope"),
        # The streaming baseline of the paper's comparison: 4 sinks + 1020 recent tokens, chunks of 256 near 128K.
        _case("window_4_1020", n=256, prev=126976, mode="window", sink=4, window=1020),
        # The 16K fold of the benchmark definition, whole: 8 chunks of 2048 tokens from an empty cache.
        _case("fold_16k", n=2048, steps=8),
        # Deep chains: chunks of 256 tokens with half of the 128K tokens folded; two steps of a chain of 511.
        _case("chain_c256_64k", n=256, steps=2, prev=65536),
        # The full-stack workload's last chunk of one layer: 4096 tokens on a cache of 124K; the largest case.
        _case("stack_c4096_128k", n=4096, prev=126976),
        # The chunk-size sweep (28 query heads on 4 KV heads) at its smallest chunk, bf16, half way.
        _case("sweep_c128_32k", hq=28, hkv=4, n=128, steps=2, prev=32768),
        # The sweep in fp32 (the precision ablation), C = 512.
        _case("sweep_f32_c512_16k", dtype="f32", hq=28, hkv=4, n=512, prev=16384),
        # The storage perturbation with the rotary embedding in the step, as a model's layer calls it: C = 1024 on 8K.
        _case("rope_int8_c1024_8k", n=1024, prev=8192, mode="rope", bits=8),
        # A model with 64-wide heads, documents chunked off any grid: 1000 tokens on 8232.
        _case("d64_c1000_8k", d=64, n=1000, prev=8232),
    ]


# Head shapes of the repository's configurations and tests: (query heads, KV heads, head dim).
_SHAPES = ((32, 8, 128), (32, 8, 128), (28, 4, 128), (32, 8, 64), (4, 1, 64), (8, 2, 128))
_MAX_TOKENS = 131072


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def _cost(case):
    """Rough seconds of a pass, for keeping drawn cases no larger than the largest listed one."""
    w = work(case)
    return max(w["flops"] / (1.4e15 if case["dtype"] == "bf16" else 1.3e14), w["bytes"] / 5e12) + 1e-5 * case["steps"] * case["layers"]


def draw(rng):
    limit = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(("decode", "question", "chunk", "chunk", "fold", "window", "rope", "storage", "f32"))
        hq, hkv, d = rng.choice(_SHAPES)
        case = dict(hq=hq, hkv=hkv, d=d, lse=rng.random() < 0.25)
        prev = _log_uniform(rng, 64, _MAX_TOKENS - 4096)
        if kind == "decode":
            case.update(n=rng.choice((1, 1, 2, 4, 8, 16)), prev=prev, layers=rng.choice((1, 2, 8)), mode=rng.choice(("plain", "noalloc", "rope")))
        elif kind == "question":
            case.update(n=rng.randint(17, 127), prev=prev, layers=rng.choice((1, 2, 4)), mode=rng.choice(("plain", "rope")))
        elif kind == "chunk":
            case.update(n=_log_uniform(rng, 128, 4096), prev=prev)
        elif kind == "fold":
            n = _log_uniform(rng, 128, 2048)
            case.update(n=n, steps=rng.randint(2, max(2, min(12, 16384 // n))), prev=0)
        elif kind == "window":
            case.update(n=_log_uniform(rng, 1, 2048), prev=prev, mode="window", sink=rng.choice((0, 4, 16)), window=_log_uniform(rng, 256, 8192))
        elif kind == "rope":
            case.update(n=_log_uniform(rng, 128, 4096), prev=prev, mode="rope")
        elif kind == "storage":
            case.update(n=_log_uniform(rng, 16, 2048), prev=prev, mode=rng.choice(("plain", "rope")), bits=rng.choice((4, 8)))
        else:
            case.update(n=_log_uniform(rng, 1, 2048), prev=min(prev, 65536), dtype="f32", mode=rng.choice(("plain", "plain", "rope")))
        case = _case(None, **case)
        if case["prev"] + case["n"] * case["steps"] <= _MAX_TOKENS and _cost(case) <= limit:
            return case


def _normal(gen, shape, dtype):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(dtype)


def prepare(case, seed):
    """Filled caches and the next chunks' q / k / v, N(0,1) as everywhere in this repository, and the output buffers."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 7919 + 20260512)
    dt = I.torch_dtype(case["dtype"])
    hq, hkv, d, n, steps, layers, prev = (case[k] for k in ("hq", "hkv", "d", "n", "steps", "layers", "prev"))
    end = prev + n * steps
    # A cache is created for its whole document and for chunks of at least 256 tokens; decoding and questions come later.
    cache = KvFoldCache(layers, hq, hkv, d, max(n, 256), max(-(-end // 1024) * 1024, 1024), case["dtype"])
    if case["bits"]:
        cache.set_storage_roundtrip(case["bits"])
    appended = []
    for layer in range(layers):
        k_rows, v_rows = cache.view(layer)
        for rows in (k_rows, v_rows):
            if prev:
                rows[:, :prev].copy_(_normal(gen, (hkv, prev, d), dt))
            new_rows = rows[:, prev:end]
            new_rows.owner = cache  # the view aliases the cache's memory: whoever holds the rows keeps the cache
            appended.append(new_rows)
    cache.set_length(-1, prev)
    q = _normal(gen, (steps, layers, n, hq, d), dt)
    k = _normal(gen, (steps, layers, n, hkv, d), dt)
    v = _normal(gen, (steps, layers, n, hkv, d), dt)
    out = torch.empty_like(q)
    lse = torch.empty((steps, layers, hq, n), device="cuda", dtype=torch.float32) if case["lse"] else None
    calls = []
    for s in range(steps):
        rope = I.rope_tables(d, prev + s * n, n, device="cuda") if case["mode"] == "rope" else None
        for layer in range(layers):
            calls.append((layer, q[s, layer], k[s, layer], v[s, layer], out[s, layer], prev + s * n,
                          lse[s, layer] if lse is not None else None, rope))
    return {"cache": cache, "prev": prev, "calls": calls, "out": out, "lse": lse, "appended": appended,
            "window": (case["sink"], case["window"]) if case["mode"] == "window" else None,
            "noalloc": case["mode"] == "noalloc", "keep": (q, k, v)}


def run(state):
    cache, window, noalloc = state["cache"], state["window"], state["noalloc"]
    cache.truncate(-1, state["prev"])
    for layer, q, k, v, out, pos, lse, rope in state["calls"]:
        cache.step(layer, q, k, v, out, pos_offset=pos, lse=lse, rope=rope, window=window, noalloc=noalloc)
    return {"out": state["out"], "lse": state["lse"], "appended": state["appended"]}


def work(case):
    """Per step and layer: the visible K and V rows of the cache, q, the new rows read and written, the output; and the
    two products over the visible (row, key) pairs."""
    es = 2 if case["dtype"] == "bf16" else 4
    hq, hkv, d, n = case["hq"], case["hkv"], case["d"], case["n"]
    total_bytes = total_flops = 0.0
    for s in range(case["steps"]):
        prev = case["prev"] + s * n
        keys, pairs = prev, n * (prev + (n + 1) / 2.0)
        if case["mode"] == "window":
            sink, window = case["sink"], case["window"]
            keys = min(prev, sink + window - 1)
            seen = [min(prev + i + 1, sink + window) for i in range(n)]
            pairs = float(sum(seen))
        total_bytes += 2.0 * hkv * d * es * (keys + 2 * n) + 2.0 * n * hq * d * es
        if case["lse"]:
            total_bytes += 4.0 * n * hq
        if case["mode"] == "rope":
            total_bytes += 4.0 * n * d
        total_flops += 4.0 * hq * d * pairs
    return {"bytes": total_bytes * case["layers"], "flops": total_flops * case["layers"]}


def tolerance(case):
    """About four times what the path differs by from the same attention in 64 bits on the stored values, measured over
    these cases and drawn ones: bf16 rel 2.5e-3 ... 3.4e-3, max 1.2e-2 (the weights and the output are rounded to 8
    bits, the queries once more after scaling); f32 rel 1.3e-6, max 6e-6 on a sample of rows (128-term dot products and
    sums over the keys in 32 bits)."""
    if case["dtype"] == "f32":
        return {"rel": 6e-6, "max": 5e-5}
    return {"rel": 1e-2, "max": 6e-2}
