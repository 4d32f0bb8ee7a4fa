"""e4m3 caches: launches on both sides of the line from which bf16 copies of the pages pay, against the oracle and, where
the copies are made, bit for bit against tiles that convert while they stage."""
import numpy as np
import pytest

import oracle
import workloads as W
from error_bar import OF_RMS, worst_of_rms
from workloads import AttnShape, make_batch

# (query lengths, context lengths, pages copied with head dim 128), 32 query heads over 2 KV heads: tiles of 16 tokens
BATCHES = {
    "few pages": ([333], [600], 38),
    "pages read 20 times": ([320], [4096 + 320], 0),                    # converted in the tiles
    "pages read 27 times": ([450], [4096 + 450], 285),
    "next to rows, few reads": ([1] * 9 + [2, 40, 17], [1, 16, 17, 300, 900, 64, 65, 2000, 31, 3000, 1500 + 40, 17], 0),
    "next to rows, many reads": ([1, 1, 450, 1], [700, 33, 4096 + 450, 1025], 285),
}


@pytest.mark.gpu
@pytest.mark.parametrize("head_dim", [128, 64])
@pytest.mark.parametrize("batch", list(BATCHES))
def test_both_sides_of_the_line(batch, head_dim):
    import gpu_harness as g
    import paper_2512_03416_amd as ts
    q, ctx, copied = BATCHES[batch]
    mk = lambda: make_batch(AttnShape(32, 2, head_dim, "bf16", "fp8"), q, ctx, seed=95, pool_rule=1.25, value_mult=1.0)
    every = sum(-(-c // 16) for n, c in zip(q, ctx) if n > 1)
    assert ts.plan_describe(g.make_desc(mk()), q, ctx).widened_pages == (copied if head_dim == 128 else every) and copied in (0, every)
    ref, rk, rv = oracle.run_batch(W.to_cpu(mk()))
    q_off = np.concatenate([[0], np.cumsum(q)])
    chunk = np.concatenate([np.arange(q_off[i], q_off[i + 1]) for i in range(len(q)) if q[i] > 1])
    for mode in (2, 1, 0) if len(q) > 1 else (2,):
        outs = []
        for options in ({}, {"prefill_widen_pages": 0})[:2 if head_dim == 128 else 1]:
            print(f"[case] {batch} D={head_dim} mode={mode} {options}", flush=True)
            # (a stated number of resident workgroups keeps so small a batch co-resident)
            out, gk, gv = g.run_batch(mk(), options={"mixed_mode": mode, "prefill_resident_workgroups": 8, **options})
            assert gk.tobytes() == rk.tobytes() and gv.tobytes() == rv.tobytes()
            assert np.all(np.isfinite(out)) and worst_of_rms(out, ref) <= OF_RMS
            outs.append(out[chunk])
        assert len(outs) == 1 or np.array_equal(outs[0], outs[1])


# prefill alone, 128 dims: (query heads, KV heads, query lengths, prefixes), pages copied
CHAINS = [((8, 8, [6000], [0]), 375), ((8, 8, [3000], [0]), 0), ((4, 4, [5896, 8716], [16, 392]), 940), ((8, 8, [4200, 4500], [0, 0]), 0),
          ((64, 8, [512], [8200]), 0)]


@pytest.mark.parametrize("batch,copied", CHAINS, ids=lambda x: str(x))
def test_long_chains_of_stages_have_their_pages_copied(batch, copied):
    """Few reads a page, but one tile's stages set the time and each of them would convert: 6000 tokens with 8/8 heads 138 us a pass
    converting, 130 with copies; 3000 (cut in two) 49 and 52."""
    import paper_2512_03416_amd as ts
    hq, hkv, q, prefix = batch
    d = ts.Desc.make(hq, hkv, 128, "bf16", "fp8", 1 << 14, 1 << 10)
    ctx = [a + b for a, b in zip(q, prefix)]
    assert ts.plan_describe(d, q, ctx).widened_pages == copied
    assert ts.plan_describe(d, q + [1] * 8, ctx + [500] * 8).widened_pages == 0      # (decode rows would wait for the copies)
