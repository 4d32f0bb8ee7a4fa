"""CPU-only checks of the boundary: exported symbols, descriptor/batch validation, planner."""
import ctypes
import os
import re

import numpy as np
import pytest

import paper_2512_03416_amd as ts
from paper_2512_03416_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "tokenscale.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(ts_[a-z_0-9]+)\s*\(", hdr))
    assert {"ts_kv_append", "ts_mixed_paged_attention", "ts_token_velocity"} <= declared
    lib = ctypes.CDLL(ts.library_path())
    for name in sorted(declared):
        assert hasattr(lib, name), name
    assert declared == set(binding.EXPORTS)


def test_library_exports_every_policy_symbol():
    from paper_2512_03416_amd import policy
    hdr = open(os.path.join(ROOT, "include", "tokenscale_policy.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(ts_[a-z_0-9]+)\s*\(", hdr))
    lib = ctypes.CDLL(ts.library_path())
    for name in sorted(declared):
        assert hasattr(lib, name), name
    assert declared == set(policy.EXPORTS)
    headers = sorted(f for f in os.listdir(os.path.join(ROOT, "include")) if f.endswith(".h"))
    assert headers == ["tokenscale.h", "tokenscale_calib.h", "tokenscale_policy.h"]   # each has a symbol test


def test_library_exports_every_calibration_symbol():
    hdr = open(os.path.join(ROOT, "include", "tokenscale_calib.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(ts_[a-z_0-9]+)\s*\(", hdr))
    lib = ctypes.CDLL(ts.library_path())
    for name in sorted(declared):
        assert hasattr(lib, name), name
    assert declared == set(binding.CALIB_EXPORTS)


def D(**kw):
    base = dict(Hq=32, Hkv=8, D=128, q_dtype="bf16", kv_dtype="bf16", num_pages=1000, max_pages_per_seq=64)
    base.update(kw)
    return ts.Desc.make(**base)


def test_check_desc_accepts_and_rejects():
    assert ts.check_desc(D()) == 0
    assert ts.check_desc(D(q_dtype="f32", kv_dtype="f32", D=64, Hq=4, Hkv=1)) == 0
    assert ts.check_desc(D(kv_dtype="fp8", Hq=64)) == 0
    assert ts.check_desc(D(page_size=32)) == binding.TS_ERR_INVALID_ARG
    assert ts.check_desc(D(Hq=30)) == binding.TS_ERR_INVALID_ARG
    assert ts.check_desc(D(num_pages=0)) == binding.TS_ERR_INVALID_ARG
    assert ts.check_desc(D(D=96)) == binding.TS_ERR_UNSUPPORTED
    assert ts.check_desc(D(q_dtype="f32", kv_dtype="bf16")) == binding.TS_ERR_UNSUPPORTED
    assert ts.check_desc(D(q_dtype=7)) == binding.TS_ERR_INVALID_ARG
    assert ts.check_desc(D(Hq=8 * 17)) == binding.TS_ERR_UNSUPPORTED


def test_cache_bytes():
    assert ts.cache_bytes(D()) == 1000 * 8 * 16 * 128 * 2
    assert ts.cache_bytes(D(kv_dtype="fp8")) == 1000 * 8 * 16 * 128
    assert ts.cache_bytes(D(q_dtype="f32", kv_dtype="f32", D=64)) == 1000 * 8 * 16 * 64 * 4
    assert ts.cache_bytes(D(D=96)) == 0


@pytest.mark.parametrize("ql,cl", [([-1], [4]), ([5], [4]), ([1], [64 * 16 + 1])])
def test_plan_rejects_bad_lengths(ql, cl):
    with pytest.raises(ts.TokenScaleError) as e:
        ts.plan_describe(D(), ql, cl)
    assert e.value.code == binding.TS_ERR_INVALID_ARG


def test_plan_counts_and_decode_items_cover_every_page_once():
    rng = np.random.default_rng(5)
    ctx = rng.integers(1, 1024, size=40)
    ql = np.ones(40, dtype=np.int32)
    ql[::7] = 0
    ql[3] = 37
    ctx[3] = 112
    ql[9] = 300
    ctx[9] = 300
    for split in (0, 8, 13, 128):
        info = ts.plan_describe(D(), ql, ctx, split)
        n_dec = int((ql == 1).sum())
        assert info.total_tokens == ql.sum() and info.decode_tokens == n_dec
        assert info.prefill_tokens == 337
        assert info.n_generic_rows == 0
        assert info.tile_tokens == 64
        assert info.n_prefill_tiles == -(-37 // 64) + -(-300 // 64)
        items = ts.plan_decode_items(D(), ql, ctx, split)
        assert len(items) == info.n_decode_items
        cover = {}
        for row, seq, n_keys, pb, pe in items:
            assert ql[seq] == 1 and n_keys == ctx[seq] and 0 <= pb < pe <= -(-n_keys // 16)
            assert pe - pb <= max(info.split_pages, 1)
            assert row == ql[:seq].sum()
            cover.setdefault(seq, []).extend(range(pb, pe))
        assert set(cover) == {s for s in range(40) if ql[s] == 1}
        for seq, pages in cover.items():
            assert sorted(pages) == list(range(-(-ctx[seq] // 16)))
        lens = items[:, 4] - items[:, 3]
        assert np.all(np.diff(lens) <= 0)                 # longest first
        n_split_rows = sum(1 for s in cover if len([1 for it in items if it[1] == s]) > 1)
        assert info.n_combine_rows == n_split_rows
        assert info.partial_slots == sum(len([1 for it in items if it[1] == s]) for s in cover
                                         if len([1 for it in items if it[1] == s]) > 1)


def test_plan_append_pages_cover_every_new_token_of_the_chunks_once():
    """Page-wise append work: each new token of a sequence with >= 8 new tokens lies in exactly one
    (page, slot range) record, and the record's row arithmetic points at that token's input row."""
    from paper_2512_03416_amd import binding
    rng = np.random.default_rng(5)
    q_lens = rng.integers(0, 70, size=60).astype(np.int32)
    q_lens[:6] = [0, 1, 7, 8, 16, 17]
    prefix = rng.integers(0, 50, size=60).astype(np.int32)
    ctx = q_lens + prefix
    desc = binding.Desc.make(8, 2, 128, "bf16", "bf16", 4096, 16)
    rec = binding.plan_export(desc, q_lens, ctx, "append")
    q_off = np.concatenate([[0], np.cumsum(q_lens)])
    seen = {}
    for seq, pg, lo, hi, row0, *_ in rec:
        assert q_lens[seq] >= 8 and 0 <= lo < hi <= 16
        for slot in range(lo, hi):
            pos = pg * 16 + slot
            assert prefix[seq] <= pos < ctx[seq]
            assert row0 + slot == q_off[seq] + pos - prefix[seq]
            assert (seq, pos) not in seen
            seen[(seq, pos)] = True
    assert len(seen) == int(q_lens[q_lens >= 8].sum())
    # the other tokens, and all tokens of shapes the page-wise kernel does not take, go one by one
    rows = binding.plan_export(desc, q_lens, ctx, "append_rows")
    want = [(q_off[s] + i, s, prefix[s] + i, 0) for s in range(len(q_lens)) if q_lens[s] < 8 for i in range(q_lens[s])]
    assert [tuple(r) for r in rows] == want
    d64 = binding.Desc.make(4, 1, 64, "f32", "f32", 4096, 16)
    assert len(binding.plan_export(d64, q_lens, ctx, "append")) == 0
    assert len(binding.plan_export(d64, q_lens, ctx, "append_rows")) == int(q_lens.sum())
    # head dim 64 with bf16 inputs is appended page-wise like head dim 128 (same lists)
    for kv in ("bf16", "fp8"):
        d64b = binding.Desc.make(8, 2, 64, "bf16", kv, 4096, 16)
        assert np.array_equal(binding.plan_export(d64b, q_lens, ctx, "append"), rec)
        assert np.array_equal(binding.plan_export(d64b, q_lens, ctx, "append_rows"), rows)


def test_plan_routes_fp32_to_generic_rows_and_head_dim_64_to_the_matrix_cores():
    d = D(q_dtype="f32", kv_dtype="f32", D=64, Hq=4, Hkv=1)
    info = ts.plan_describe(d, [1, 37, 64], [5, 37, 112])
    assert info.n_generic_rows == 102 and info.n_decode_items == 0 and info.n_prefill_tiles == 0
    # head dim 64, bf16 cache: decode rows are matrix-core items, chunks matrix-core tiles, one launch per class
    info = ts.plan_describe(D(D=64), [1, 4], [5, 4])
    assert info.n_generic_rows == 0 and info.n_decode_items == 1 and info.n_prefill_tiles == 1 and info.mixed_mode == 0
    # head dim 64, e4m3 cache: the tiles read widened pages; without them the chunk rows take the generic kernel
    info = ts.plan_describe(D(D=64, kv_dtype="fp8"), [1, 1, 40], [5, 1000, 17 + 40])
    assert info.n_generic_rows == 0 and info.n_decode_items >= 2 and info.n_prefill_tiles >= 1 and info.widened_pages == 4
    rows = binding.plan_export(D(D=64, kv_dtype="fp8", max_pages_per_seq=20000), [40], [40 + 16 * 16384], "rows")
    assert len(rows) == 40                                    # more pages than the widening scratch takes


def test_plan_sizes_the_co_resident_launch_from_the_two_costs():
    """A mixed batch is launched co-resident with as many resident prefill workgroups as the ratio of the two
    classes' estimated times asks for (all CUs when the tiles take about as long as the scan or longer, fewer -- in
    multiples of the die count -- when the decode scan outlasts them); a batch in which either class is short goes class by class."""
    rng = np.random.default_rng(3)
    dec = rng.integers(1024, 8193, 128).tolist()
    d = D(max_pages_per_seq=2048, num_pages=200000)

    def plan(chunks):
        q = [1] * len(dec) + [c for c, _ in chunks]
        ctx = dec + [c + p for c, p in chunks]
        return ts.plan_describe(d, q, ctx)
    # tiles about as long as a scan of 150 us or more: all CUs (with fewer the rows on CUs of their own, four workgroups to a
    # CU, end last: 585 us a pass with 256, 640 with 192)
    burst = plan([(2048, 0), (2048, 1500), (2048, 3000), (2048, 4096)])
    assert burst.mixed_mode == 2 and burst.prefill_workgroups == 256
    heavy = plan([(4096, 4096)] * 4)                                                 # tiles dominate
    assert heavy.mixed_mode == 2 and heavy.prefill_workgroups == 256
    one = plan([(1920, 4096)])                                                       # the scan dominates
    assert one.mixed_mode == 2 and 64 <= one.prefill_workgroups <= 160 and one.prefill_workgroups % 8 == 0
    small = plan([(384, 4096)])
    assert small.mixed_mode == 2 and 8 <= small.prefill_workgroups <= 96
    assert plan([(128, 0)]).mixed_mode == 0 and plan([(128, 0)]).prefill_workgroups == 0
    few = ts.plan_describe(d, [1, 1, 2048], [100, 200, 2048])                        # hardly any decode pages
    assert few.mixed_mode == 0 and few.prefill_workgroups == 0
    # monotone in the prefill work
    sizes = [plan([(n, 4096)]).prefill_workgroups for n in (512, 1024, 2048, 4096, 8192)]
    assert sizes == sorted(sizes) and sizes[-1] == 256


def test_create_without_gpu_fails_loudly():
    import torch
    if torch.cuda.is_available():
        pytest.skip("GPU present")
    with pytest.raises(ts.TokenScaleError) as e:
        ts.Context(D())
    assert e.value.code == binding.TS_ERR_HIP


def test_calibration_helpers_reject_bad_arguments_before_touching_a_gpu():
    lib = binding.load_library()
    flops = ctypes.c_int64(-1)
    one = ctypes.c_void_p(16)                                  # never dereferenced: the checks come first
    assert lib.ts_calib_mfma(None, None, one, 10, 0, ctypes.byref(flops)) == -1
    assert lib.ts_calib_mfma(None, one, None, 10, 0, ctypes.byref(flops)) == -1
    assert lib.ts_calib_mfma(None, one, one, 0, 0, ctypes.byref(flops)) == -1
    assert lib.ts_calib_mfma(None, one, one, 200001, 1, ctypes.byref(flops)) == -1
    assert lib.ts_calib_mfma(None, one, one, 10, 1, None) == -1
    assert flops.value == -1
    assert lib.ts_calib_copy(None, one, one, 24) == -1         # not a multiple of 16
    assert lib.ts_calib_read(None, one, None, 32) == -1


@pytest.mark.parametrize("seed", range(6))
def test_plan_invariants_on_seeded_random_batches(seed):
    """Every list of the planner against what the batch demands, for random mixes of empty sequences,
    decode rows and chunks: each cache page of a decode row in exactly one item, partial slots
    contiguous per split row, each chunk token in exactly one tile, each (tile, head) once in the launch
    order and once in the queues, each (decode item, head) once in the queues, append work covering each
    new token once."""
    rng = np.random.default_rng(4000 + seed)
    hkv = int(rng.choice([1, 2, 8]))
    group = int(rng.choice([1, 4, 8]))
    desc = binding.Desc.make(hkv * group, hkv, 128, "bf16", str(rng.choice(["bf16", "fp8"])), 1 << 16, 1024)
    n = int(rng.integers(1, 40))
    kinds = rng.choice(["empty", "decode", "decode", "chunk"], size=n)
    ql = np.array([0 if k == "empty" else 1 if k == "decode" else int(rng.integers(2, 900)) for k in kinds], dtype=np.int32)
    ctx = ql + rng.integers(0, 6000, size=n).astype(np.int32)
    split = int(rng.choice([0, 0, 8, 37]))
    slots = int(rng.choice([0, 96, 768]))
    mode = int(rng.choice([-1, 0, 1, 2]))
    exp = lambda which: binding.plan_export(desc, ql, ctx, which, split, slots, mode)
    q_off = np.concatenate([[0], np.cumsum(ql)])
    pages = -(-ctx // 16)
    tile_tokens = 256 // group

    dec, cmb = exp("decode"), exp("combine")
    cover, slots_of = {}, {}
    for row, seq, n_keys, pb, pe, part, *_ in dec:
        assert ql[seq] == 1 and row == q_off[seq] and n_keys == ctx[seq] and 0 <= pb < pe <= pages[seq]
        cover.setdefault(seq, []).extend(range(pb, pe))
        slots_of.setdefault(seq, []).append(part)
    assert set(cover) == {s for s in range(n) if ql[s] == 1}
    for s, pg in cover.items():
        assert sorted(pg) == list(range(pages[s]))
    split_rows = {s for s, p in slots_of.items() if len(p) > 1}
    assert all(p == [-1] for s, p in slots_of.items() if s not in split_rows)
    used = []
    assert len(cmb) == len(split_rows)
    for row, begin, n_split, _ in cmb:
        s = int(np.searchsorted(q_off, row, side="right") - 1)
        while ql[s] == 0:
            s += 1
        assert s in split_rows and sorted(slots_of[s]) == list(range(begin, begin + n_split))
        used.extend(range(begin, begin + n_split))
    assert sorted(used) == list(range(len(used)))

    pf = exp("prefill")
    toks, part_keys = {}, {}
    for seq, row0, q_len, prefix, t0, cnt, ctx_len, part, kv_b, kv_e, *_ in pf:
        assert ql[seq] > 1 and row0 == q_off[seq] and q_len == ql[seq] and prefix == ctx[seq] - ql[seq] and ctx_len == ctx[seq]
        assert t0 % tile_tokens == 0 and 0 < cnt <= tile_tokens
        hi = prefix + t0 + cnt                                    # keys the tile's last row sees
        if part < 0:
            assert kv_b == 0 and kv_e >= hi
            toks.setdefault(seq, []).extend(range(t0, t0 + cnt))
        else:                                                     # a part of a tile cut along the keys
            assert kv_b % 64 == 0 and kv_b <= prefix + t0 and kv_b < min(kv_e, hi)
            assert kv_e % 64 == 0 or kv_e >= hi
            part_keys.setdefault((seq, t0, cnt), []).append((kv_b, min(kv_e, hi), part))
    for (seq, t0, cnt), parts in part_keys.items():               # the parts of a tile cover its keys exactly once
        parts.sort()
        assert len(parts) > 1 and parts[0][0] == 0 and parts[-1][1] == ctx[seq] - ql[seq] + t0 + cnt
        assert all(a[1] == b[0] for a, b in zip(parts, parts[1:]))
        assert all(e <= ctx[seq] - ql[seq] + t0 for _, e, _ in parts[:-1])        # only the last part meets the diagonal
        assert [p for _, _, p in parts] == list(range(parts[0][2], parts[0][2] + len(parts)))
        toks.setdefault(seq, []).extend(range(t0, t0 + cnt))
    pfc = exp("pfcombine")
    assert len(pfc) == len(part_keys)
    for item, p0, n_part, _ in pfc:
        seq, _, _, _, t0, cnt, *_ = pf[item]
        assert len(part_keys[(seq, t0, cnt)]) == n_part and min(p for _, _, p in part_keys[(seq, t0, cnt)]) == p0
    assert set(toks) == {s for s in range(n) if ql[s] > 1}
    for s, t in toks.items():
        assert sorted(t) == list(range(ql[s]))

    pfmap = exp("pfmap")
    live = [(int(t), int(g)) for t, g in pfmap if t >= 0]
    assert sorted(live) == sorted((t, g) for t in range(len(pf)) for g in range(hkv))      # (every part is a work item)

    queue, qoff = exp("queue"), exp("qoff")[:, 0]
    if len(dec) and len(pf) and mode == 1:
        assert len(queue)                                     # (asked for by name: no other launch form is chosen)
    if len(dec) and len(pf) and mode != 0 and len(queue):     # a mixed batch has per-die queues, unless the planner
        assert len(qoff) == 9 and qoff[0] == 0 and qoff[-1] == len(queue) and np.all(np.diff(qoff) >= 0)
        d_entries = sorted((int(i), int(g)) for k, i, g, _ in queue if k == 0)
        p_entries = sorted((int(i), int(g)) for k, i, g, _ in queue if k == 1)
        # launches it class by class (either class too short for the co-resident launch to pay).
        # One persistent kernel: both kinds are queued; co-resident launch: the tiles only
        assert d_entries in ([], sorted((i, g) for i in range(len(dec)) for g in range(hkv)))
        assert mode != 1 or d_entries
        assert p_entries == sorted((t, g) for t in range(len(pf)) for g in range(hkv))
    else:
        assert len(queue) == 0

    seen = set()
    for seq, pg, lo, hi, row0, *_ in exp("append"):
        for slot in range(lo, hi):
            pos = pg * 16 + slot
            assert (seq, pos) not in seen and row0 + slot == q_off[seq] + pos - (ctx[seq] - ql[seq])
            seen.add((seq, pos))
    for row, seq, pos, _ in exp("append_rows"):
        assert (seq, pos) not in seen and row == q_off[seq] + pos - (ctx[seq] - ql[seq])
        seen.add((seq, pos))
    assert seen == {(s, p) for s in range(n) for p in range(ctx[s] - ql[s], ctx[s])}


@pytest.mark.parametrize("q_lens,ctx_lens", [(5, 9), (np.int64(5), np.array(9)), ([5], (9,)), ([5, 0, 1], np.array([9, 3, 4])),
                                             (np.array([5, 1, 7, 1])[::2], np.array([9, 8], np.uint8)), ([], []),
                                             (np.array([5.0, 1.0]), [9, 4])])
def test_binding_takes_lengths_in_every_form(q_lens, ctx_lens):
    """Lengths reach the library as int32 arrays of as many sequences: a single number, lists, arrays of any integer type
    and stride, none at all."""
    calls = []

    class Library:
        def __getattr__(self, name):
            return lambda *args: calls.append((name, args)) or 0
    ctx = binding.Context.__new__(binding.Context)
    ctx._lib, ctx._h = Library(), ctypes.c_void_p(1)
    ctx.kv_append(None, None, None, None, None, None, None, q_lens, ctx_lens, stream=0)
    for noalloc in (False, True):
        ctx.mixed_paged_attention(None, None, None, None, None, None, None, None, q_lens, ctx_lens, 0.0, None, stream=0,
                                  noalloc=noalloc)
    ctx._h = None
    want_q, want_c = (np.atleast_1d(np.asarray(x)).astype(np.int32) for x in (q_lens, ctx_lens))
    assert [c[0] for c in calls[:3]] == ["ts_kv_append", "ts_mixed_paged_attention", "ts_mixed_paged_attention_noalloc"]
    for _, args in calls[:3]:
        at = next(i for i, x in enumerate(args) if isinstance(x, bytes))
        assert np.array_equal(np.frombuffer(args[at], np.int32), want_q)
        assert np.array_equal(np.frombuffer(args[at + 1], np.int32), want_c)
        assert args[at + 2] == len(want_q)


def test_whole_decode_rows_are_packed_in_little_host_time():
    """Rows that come out even over the CUs stay whole (a plain longest-first packing says when), and deciding so costs a
    batch of 700 rows on 256 CUs no more host time than planning 800 rows that are not packed (with room for noise)."""
    import heapq
    import time
    rng = np.random.default_rng(11)
    whole = 0
    for kv_heads, lo, hi in [(8, 100, 400), (8, 300, 900), (4, 16, 700), (2, 16, 300), (1, 16, 200), (3, 50, 600)] * 6:
        desc = ts.Desc.make(4 * kv_heads, kv_heads, 128, "bf16", "bf16", 1 << 20, 256)
        cus = 256 // kv_heads
        n = int(rng.integers(cus, 768 // kv_heads + 1))
        ctx = rng.integers(lo, hi + 1, n)
        pages = sorted(((int(c) + 15) // 16 + 4 for c in ctx), reverse=True)         # 4: what an item costs
        room, heap = -(-n // cus), [(0, b, 0) for b in range(cus)]
        longest = 0
        for p in pages:
            load, b, k = heapq.heappop(heap)
            longest = max(longest, load + p)
            if k + 1 < room:
                heapq.heappush(heap, (load + p, b, k + 1))
        if longest <= sum(pages) // cus + 24:
            whole += 1
            info = ts.plan_describe(desc, np.ones(n, np.int32), ctx)
            assert info.n_decode_items == n and info.n_combine_rows == 0
    assert whole > 12

    desc = ts.Desc.make(4, 1, 128, "bf16", "bf16", 1 << 20, 256)

    def host_time(n):
        q, ctx = np.ones(n, np.int32), rng.integers(16, 201, n).astype(np.int32)
        best = 1.0
        for _ in range(300):
            t = time.perf_counter()
            ts.plan_describe(desc, q, ctx)
            best = min(best, time.perf_counter() - t)
        return best
    assert host_time(700) <= 2.0 * host_time(800)


@pytest.mark.parametrize("mode,kv_heads", [(1, 8), (2, 8), (1, 70000), (2, 70000)])
def test_queues_hold_every_item_of_every_kv_head(mode, kv_heads):
    """The per-die queues name each (decode item, KV head) and (prefill tile, KV head) pair once, whatever the number of
    KV heads (mode 2: the tiles only)."""
    desc = ts.Desc.make(kv_heads, kv_heads, 128, "bf16", "bf16", 4096, 512)
    ql, cl = ([1] * 64 + [2048], [4096] * 65) if kv_heads == 8 else ([1, 300], [4096, 1024])
    queue = ts.plan_export(desc, ql, cl, "queue", mixed_mode=mode)
    assert len(queue) > 0
    want = set()
    for kind, name in ((0, "decode"), (1, "prefill")):
        if kind == 1 or mode == 1:
            n = len(ts.plan_export(desc, ql, cl, name, mixed_mode=mode))
            want |= {(kind, i, g) for i in range(n) for g in range(kv_heads)}
    got = [tuple(int(x) for x in r[:3]) for r in queue]
    assert len(got) == len(want) and set(got) == want


@pytest.mark.parametrize("lens,longest_first", [([512, 128, 300, 130, 444, 257, 65, 2], True), ([64] * 16, True),
                                                ([1024] * 8, False), ([300] * 24, False)])
def test_launch_order_of_few_prompts(lens, longest_first):
    """A die with at most two tiles per CU takes them longest first; with more, one (chunk, KV head) stream after the
    other.  Either way every (tile, head) is launched once and a stream stays on one die."""
    desc = ts.Desc.make(32, 8, 128, "bf16", "bf16", 4096, 128)
    pf = ts.plan_export(desc, lens, lens, "prefill")
    pfmap = ts.plan_export(desc, lens, lens, "pfmap")
    live = [(int(t), int(g)) for t, g in pfmap if t >= 0]
    assert sorted(live) == sorted((t, g) for t in range(len(pf)) for g in range(8))
    home = {}
    for x in range(8):
        die = [(int(t), int(g)) for t, g in pfmap[x::8] if t >= 0]
        keys = [pf[t][3] + pf[t][4] + pf[t][5] for t, _ in die]
        streams = [(int(pf[t][0]), g) for t, g in die]
        for st in streams:
            assert home.setdefault(st, x) == x
        if longest_first:
            assert keys == sorted(keys, reverse=True)
        else:
            assert len([1 for a, b in zip([None] + streams, streams) if a != b]) == len(set(streams))


def test_kernels_fit_their_register_budget_without_spilling():
    """The co-resident launch rests on register budgets: resident prefill workgroups at <= 192 vector registers
    per lane (two waves per SIMD) next to a lean decode workgroup at <= 128, and no kernel may spill (a spill
    reload waits for every load in flight, the stage copies included).  Compiles the kernel sources for gfx950
    with the library's flags and reads the compiler's resource remarks."""
    import subprocess
    from paper_2512_03416_amd import build as B
    budgets = {"prefill_resident_kernel": 192, "prefill_kernel": 192, "decode_kernel_lean": 128, "mixed_kernel": 256,
               "decode_kernel": 256, "row_tile_kernel": 256}
    seen = set()
    for src in ("ts_kernels_mixed.hip", "ts_kernels_prefill.hip", "ts_kernels_decode.hip", "ts_kernels_rows.hip",
                "ts_kernels_append.hip"):
        r = subprocess.run([B.HIPCC] + B.FLAGS + ["-Rpass-analysis=kernel-resource-usage", "-x", "hip", "-c",
                                                 os.path.join(B.CSRC, src), "-o", os.devnull],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        name = None
        for line in r.stderr.splitlines():
            m = re.search(r"Function Name: (\S+)", line)
            if m:
                name = m.group(1)
            m = re.search(r" VGPRs: (\d+)", line)
            if m and name:
                key = next((k for k in sorted(budgets, key=len, reverse=True) if k in name), None)
                if key:
                    assert int(m.group(1)) <= budgets[key], (name, line)
                    seen.add(key)
            m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
            if m and name:
                assert int(m.group(1)) == 0, f"{name} uses scratch memory (spills)"
    assert seen == set(budgets)
