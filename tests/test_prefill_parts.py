"""How prefill tiles are cut along the keys: every key once, cuts on stages that all rows see, four parts before more."""
import numpy as np
import pytest

import oracle
import workloads as W
from error_bar import OF_RMS, worst_of_rms
from workloads import AttnShape, make_batch


@pytest.mark.parametrize("heads", [(32, 8), (64, 8), (4, 1)], ids=lambda h: f"{h[0]}q{h[1]}kv")
def test_cut_tiles_cover_their_keys_once(heads):
    import paper_2512_03416_amd as ts
    from paper_2512_03416_amd import binding
    d = ts.Desc.make(heads[0], heads[1], 128, "bf16", "bf16", 1 << 14, 1 << 10)
    for prefix in [0, 63, 64, 448, 511, 512, 767, 768, 831, 1000, 1024, 1500, 2047, 2048, 2560, 3071, 3072, 3500, 4096, 9000]:
        tiles = binding.plan_export(d, [40], [prefix + 40], "prefill")
        by_tile = {}
        for t in tiles:
            by_tile.setdefault(int(t[4]), []).append((int(t[8]), int(t[9])))
        for tok, ranges in by_tile.items():
            ranges.sort()
            assert ranges[0][0] == 0 and ranges[-1][1] == 2**31 - 1
            for (_, end), (begin, _) in zip(ranges, ranges[1:]):
                assert end == begin and begin % 64 == 0 and 0 < begin <= prefix + tok
            below = (prefix + tok) // 64 * 64
            launch = (prefix + max(by_tile)) // 64 * 64 >= 6 * 512              # (a merge is launched: all tiles in whole ranges)
            least = 1024 if launch else 768
            most = 16 if launch else 4 if below >= 768 else 1
            assert len(ranges) <= most and (len(ranges) > 1) == (below >= least), (prefix, tok, ranges)


# (query heads, KV heads, cache, chunks, prefixes), parts of the tiles in query order, sequence by sequence
HALVES = {
    "a merge is launched for another tile": ((32, 8, "fp8", [7, 30, 20], [2645, 5403, 4000]), [[5], [10], [7]]),
    "more pieces than a die has CUs, few KV heads": ((64, 4, "bf16", [106, 339], [993, 993]), [[1] * 2 + [2] * 5, [1] * 2 + [2] * 20]),
    "the same, one chunk": ((16, 2, "bf16", [160, 160], [800, 800]), [[3, 3, 3, 3, 3]] * 2),
    "the same, one longer chunk": ((16, 2, "bf16", [900], [800]), [[1] * 7 + [2] * 16 + [3] * 6]),
    "nearly a tile per CU, bf16": ((32, 8, "bf16", [300, 294, 327], [900, 885, 1026]), [[1, 1, 2, 2, 2], [1, 1, 1, 2, 2], [2] * 6]),
    "nearly a tile per CU, e4m3": ((32, 8, "fp8", [300, 294, 327], [900, 885, 1026]), [[2] * 5, [2] * 5, [2] * 6]),
    "a prompt of varied tiles, few KV heads": ((8, 4, "bf16", [1400], [0]), [[1] * 6 + [3, 3, 4, 4, 4]]),
    "ranges would come to a launch": ((4, 2, "bf16", [1700], [1400]), [[4] * 14]),
}


@pytest.mark.parametrize("case", list(HALVES))
def test_halves_of_the_shortest_range_only_where_they_pay(case):
    from paper_2512_03416_amd import binding
    import paper_2512_03416_amd as ts
    (hq, hkv, kv, q, prefix), want = HALVES[case]
    d = ts.Desc.make(hq, hkv, 128, "bf16", kv, 1 << 14, 1 << 10)
    got = [{} for _ in q]
    for t in binding.plan_export(d, q, [a + b for a, b in zip(q, prefix)], "prefill"):
        got[int(t[0])][int(t[4])] = got[int(t[0])].get(int(t[4]), 0) + 1
    assert [[g[t] for t in sorted(g)] for g in got] == want


@pytest.mark.gpu
@pytest.mark.parametrize("kv,heads,head_dim", [("bf16", (8, 2), 128), ("fp8", (16, 2), 128), ("bf16", (8, 2), 64)])
@pytest.mark.parametrize("prefix", [767, 768, 1100, 2047, 3071, 3072])
def test_short_chunks_over_prefixes_of_a_few_parts(kv, heads, head_dim, prefix):
    import gpu_harness as g
    mk = lambda: make_batch(AttnShape(heads[0], heads[1], head_dim, "bf16", kv), [70], [prefix + 70], seed=97, pool_rule=1.25, value_mult=0.5)
    ref, rk, rv = oracle.run_batch(W.to_cpu(mk()))
    print(f"[case] kv={kv} heads={heads} D={head_dim} prefix={prefix}", flush=True)
    out, gk, gv = g.run_batch(mk())
    assert gk.tobytes() == rk.tobytes() and gv.tobytes() == rv.tobytes()
    assert np.all(np.isfinite(out)) and worst_of_rms(out, ref) <= OF_RMS
