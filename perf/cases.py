"""Performance cases of the mixed paged-attention pass: what a serving loop has the library do.

A case is a batch of one serving iteration -- decode rows (one new token each), prefill chunks, or both -- over a
paged cache that already holds the sequences' earlier tokens.  `prepare` makes what a serving process has in hand
before the call: the context of the layer (with its scratch reserved), the two caches filled through the library's
own append, the page table, and the iteration's queries and new K/V rows.  `run` is one call of the pass (or of the
append alone, for prompts whose K/V arrive from a prefill instance).

Lengths are drawn from the case's own `lengths` seed, so a case is the same batch whatever the inputs' seed;
values are normal, page tables random permutations of the pool.
"""
import math

import numpy as np
import torch

import paper_2512_03416_amd as ts

PAGE = 16
_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}
_SIZE = {"f32": 4, "bf16": 2, "fp8": 1}


def _case(name, heads, dtype, cache, rows=0, ctx=(0, 0), dist="uniform", chunks=0, chunk=(0, 0), prefix=(0, 0),
          entry="pass", lengths=1):
    """rows decode rows with a context in ctx (uniform, or lognormal around the geometric middle), then `chunks`
    prefill chunks of `chunk` tokens over a cached `prefix`; entry: "pass", "noalloc" (the pass without allocation)
    or "append"."""
    c = {"q_heads": heads[0], "kv_heads": heads[1], "head_dim": heads[2], "dtype": dtype, "cache": cache,
         "rows": rows, "ctx_lo": ctx[0], "ctx_hi": ctx[1], "ctx_dist": dist, "chunks": chunks, "chunk_lo": chunk[0],
         "chunk_hi": chunk[1], "prefix_lo": prefix[0], "prefix_hi": prefix[1], "entry": entry, "lengths": lengths}
    return dict(c, name=name) if name else c


def listed():
    gqa4, gqa5, gqa8 = (32, 8, 128), (40, 8, 128), (64, 8, 128)
    return [
        # The smallest pass: a handful of short sequences in full precision; latency and launches are all of it.
        _case("tiny_mixed_f32", (4, 1, 64), "f32", "f32", 6, (1, 200), chunks=2, chunk=(37, 64), prefix=(0, 48)),
        # A full-precision layer serving a small mixed batch (reference runs, precision studies).
        _case("mixed_f32", gqa4, "f32", "f32", 16, (64, 2048), chunks=1, chunk=(231, 231), prefix=(300, 300)),
        # A decoder at low load: few rows of ordinary length, one launch-bound pass per token.
        _case("decode_few_bf16", gqa4, "bf16", "bf16", 8, (500, 2500)),
        # Head dim 64, a decoder at medium load.
        _case("decode_hd64_bf16", (32, 8, 64), "bf16", "bf16", 48, (200, 6000)),
        # A full decode batch: the scan of the whole cache that sets the time per output token.
        _case("decode_batch_bf16", gqa4, "bf16", "bf16", 256, (512, 4096)),
        # Few requests with very long contexts, e4m3 cache.
        _case("decode_long_fp8", gqa8, "bf16", "fp8", 3, (30000, 131072)),
        # The first step of chunked prefill over a set of waiting prompts, ragged, nothing cached yet.
        _case("prefill_prompts_bf16", gqa4, "bf16", "bf16", chunks=8, chunk=(128, 512)),
        # One restricted chunk of a long prompt, deep in its own prefix.
        _case("prefill_prefix_fp8", gqa8, "bf16", "fp8", chunks=1, chunk=(512, 512), prefix=(8200, 8200)),
        # An ordinary iteration of a decoder that absorbs prefill: some decode rows and one chunk that fills the
        # profiled chunk size.
        _case("mixed_absorb_bf16", gqa5, "bf16", "bf16", 24, (300, 3000), chunks=1, chunk=(2024, 2024),
              prefix=(1000, 1000)),
        # A burst on a loaded decoder: long decode rows next to several chunks over cached prefixes.
        _case("mixed_burst_bf16", gqa4, "bf16", "bf16", 128, (1024, 8192), chunks=4, chunk=(2048, 2048),
              prefix=(0, 4096)),
        # The largest: a 70B-like layer with an e4m3 cache, a large heavy-tailed decode batch and 64 Ki prompt tokens.
        _case("mixed_burst_fp8", gqa8, "bf16", "fp8", 512, (256, 32768), "lognormal", chunks=16, chunk=(4096, 4096)),
        # K/V of finished prompts arriving from a prefill instance: the append alone.
        _case("append_prompts_bf16", gqa4, "bf16", "bf16", chunks=12, chunk=(100, 4000), entry="append"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A batch of the same ranges: kinds, types and geometries as listed, sizes over the whole range."""
    while True:
        kind = rng.choice(["decode", "decode", "prefill", "mixed", "mixed", "append"])
        dtype, cache = rng.choice([("bf16", "bf16")] * 3 + [("bf16", "fp8")] * 2 + [("f32", "f32")])
        full = dtype == "f32"
        heads = rng.choice([(4, 1, 64), (32, 8, 64), (32, 8, 128)] if full else
                           [(32, 8, 128), (32, 8, 128), (40, 8, 128), (64, 8, 128), (32, 8, 64)])
        c = _case("", heads, dtype, cache, lengths=rng.randrange(1 << 16))
        if kind in ("decode", "mixed"):
            c["rows"] = _log(rng, 1, 32 if full else 512)
            c["ctx_hi"] = _log(rng, 16, 2048 if full else 131072)
            c["ctx_lo"] = max(1, int(c["ctx_hi"] * rng.uniform(0.1, 0.9)))
            c["ctx_dist"] = rng.choice(["uniform", "lognormal"])
        if kind != "decode":
            c["chunks"] = _log(rng, 1, 3 if full else 16)
            c["chunk_hi"] = _log(rng, 16, 300 if full else 4096)
            c["chunk_lo"] = max(2, int(c["chunk_hi"] * rng.uniform(0.1, 1.0)))
            c["prefix_hi"] = rng.choice([0, _log(rng, 16, 500 if full else 16384)])
            c["prefix_lo"] = int(c["prefix_hi"] * rng.uniform(0.0, 1.0))
        if kind == "append":
            c["entry"] = "append"
        elif kind == "decode" and c["rows"] <= 64 and c["rows"] * c["ctx_hi"] <= 64000 and rng.random() < 0.25:
            c["entry"] = "noalloc"
        w = work(c)
        ctx = _lengths(c)[1].astype(np.int64)
        if full and w["flops"] <= 1.8e9:
            return c
        if not full and w["flops"] <= 4e12 and w["bytes"] <= 6e9 and ctx.sum() <= 3 << 20 and ctx[c["rows"]:].sum() <= 200000:
            return c


def _lengths(c):
    """(q_lens, ctx_lens): decode rows first, then the chunks."""
    rng = np.random.default_rng(c["lengths"])
    n = c["rows"]
    if c["ctx_dist"] == "lognormal" and n:
        med = math.sqrt(c["ctx_lo"] * c["ctx_hi"])
        dec = np.clip(np.rint(np.exp(math.log(med) + 0.8 * rng.standard_normal(n))), c["ctx_lo"], c["ctx_hi"])
    else:
        dec = rng.integers(c["ctx_lo"], c["ctx_hi"] + 1, n)
    q = rng.integers(c["chunk_lo"], c["chunk_hi"] + 1, c["chunks"])
    p = rng.integers(c["prefix_lo"], c["prefix_hi"] + 1, c["chunks"])
    q_lens = np.concatenate([np.ones(n, np.int64), q])
    return q_lens.astype(np.int32), (np.concatenate([dec.astype(np.int64), p + q])).astype(np.int32)


def _randn(gen, rows, heads, dim, dtype):
    return torch.randn((rows, heads, dim), generator=gen, device="cuda", dtype=_TORCH[dtype])


def prepare(case, seed):
    q_lens, ctx_lens = _lengths(case)
    prefix = (ctx_lens - q_lens).astype(np.int32)
    pages = (ctx_lens.astype(np.int64) + PAGE - 1) // PAGE
    hq, hkv, dim, dtype = case["q_heads"], case["kv_heads"], case["head_dim"], case["dtype"]
    pool = int(math.ceil(1.25 * pages.sum()))                   # a quarter of the pool is free
    width = int(pages.max())
    perm = np.random.default_rng(seed).permutation(pool).astype(np.int32)
    table = np.full((len(q_lens), width), -1, np.int32)
    at = 0
    for s, n in enumerate(pages):
        table[s, :n] = perm[at:at + n]
        at += n
    desc = ts.Desc.make(hq, hkv, dim, dtype, case["cache"], pool, width)
    ctx = ts.Context(desc)
    total = int(q_lens.sum())
    ctx.reserve(total, len(q_lens), int(pages.sum()))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    k_cache = torch.zeros(ts.cache_bytes(desc), dtype=torch.uint8, device="cuda")
    v_cache = torch.zeros_like(k_cache)
    k_scale = v_scale = None
    if case["cache"] == "fp8":                                  # calibrated per head, about 4.5 standard deviations
        k_scale, v_scale = ((4.0 + torch.rand(hkv, generator=gen, device="cuda")) / 448.0 for _ in range(2))
    table_dev = torch.from_numpy(table).cuda()
    # the sequences' earlier tokens, in groups that bound the memory their K/V rows take on the way
    s = 0
    while s < len(q_lens):
        e, n = s, 0
        while e < len(q_lens) and (e == s or n + int(prefix[e]) <= 1 << 19):
            n += int(prefix[e])
            e += 1
        if n:
            k, v = _randn(gen, n, hkv, dim, dtype), _randn(gen, n, hkv, dim, dtype)
            ctx.kv_append(k, v, k_cache, v_cache, k_scale, v_scale, table_dev[s:e], prefix[s:e], prefix[s:e])
        s = e
    q = _randn(gen, total, hq, dim, dtype)
    k_new, v_new = _randn(gen, total, hkv, dim, dtype), _randn(gen, total, hkv, dim, dtype)
    return {"ctx": ctx, "q": q, "k": k_new, "v": v_new, "k_cache": k_cache, "v_cache": v_cache, "k_scale": k_scale,
            "v_scale": v_scale, "table": table_dev, "q_lens": q_lens, "ctx_lens": ctx_lens, "out": torch.empty_like(q),
            "entry": case["entry"]}


def run(state):
    s = state
    if s["entry"] == "append":
        s["ctx"].kv_append(s["k"], s["v"], s["k_cache"], s["v_cache"], s["k_scale"], s["v_scale"], s["table"],
                           s["q_lens"], s["ctx_lens"])
        return {"k_cache": s["k_cache"], "v_cache": s["v_cache"]}
    s["ctx"].mixed_paged_attention(s["q"], s["k"], s["v"], s["k_cache"], s["v_cache"], s["k_scale"], s["v_scale"],
                                   s["table"], s["q_lens"], s["ctx_lens"], 0.0, s["out"],
                                   noalloc=s["entry"] == "noalloc")
    return {"out": s["out"], "k_cache": s["k_cache"], "v_cache": s["v_cache"]}


def work(case):
    """Bytes: earlier tokens' K/V read, new K/V rows read and stored, queries read, outputs written, page ids.
    Flops: two products over every key that a row sees."""
    q_lens, ctx_lens = (a.astype(np.int64) for a in _lengths(case))
    prefix = ctx_lens - q_lens
    row, kv_row = case["q_heads"] * case["head_dim"], 2 * case["kv_heads"] * case["head_dim"]
    es, cs, total = _SIZE[case["dtype"]], _SIZE[case["cache"]], int(q_lens.sum())
    nbytes = total * kv_row * (es + cs) + 4 * int(((ctx_lens + PAGE - 1) // PAGE).sum())
    if case["entry"] == "append":
        return {"bytes": nbytes, "flops": 0}
    nbytes += int(prefix.sum()) * kv_row * cs + total * row * 2 * es
    keys = int((q_lens * prefix + q_lens * (q_lens + 1) // 2).sum())
    return {"bytes": nbytes, "flops": 4 * row * keys}


def tolerance(case):
    if case["entry"] == "append":
        return "exact"                                          # cache bytes
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 2e-5}                       # against 64 bits: up to 5.4e-7, 5.1e-6
    return {"rel": 1e-2, "max": 6e-2}                           # (bf16 weights and outputs) up to 2.4e-3, 2.1e-2
