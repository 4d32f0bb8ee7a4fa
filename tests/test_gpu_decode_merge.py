"""The end of a decode item: its waves' states added up by all threads, in halves of eight heads or at once; the chunks
of split rows added up two at a time or one."""
import numpy as np
import pytest

import oracle
import workloads as W
from error_bar import OF_RMS, worst_of_rms
from workloads import AttnShape, make_batch

pytestmark = pytest.mark.gpu

# of items of 8 pages: 1, 2, 8, 9, 16, 17, 24, 25 (whole chunks of eight partials, odd and even numbers of them, with one left)
CTX = [1, 17, 128, 129, 1024, 1025, 2048, 2049, 3072, 3073]
FORMS = [{}, {"decode_split_pages": 8, "decode_merge_in_kernel": 1}, {"decode_split_pages": 8, "decode_merge_in_kernel": 0},
         {"decode_split_pages": 8, "decode_merge_in_kernel": 1, "decode_fused_append": 0}, {"decode_prefetch_tiles": 3}]
MIXED = [{"mixed_mode": m, "decode_split_pages": s} for m in (0, 1) for s in (0, 8)]


@pytest.mark.parametrize("head_dim", [128, 64])
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("heads", [(1, 1), (8, 1), (9, 1), (15, 1), (32, 2)], ids=lambda h: f"{h[0]}q{h[1]}kv")
def test_every_form_of_the_merge_against_the_oracle(kv, heads, head_dim):
    import gpu_harness as g
    shape = AttnShape(heads[0], heads[1], head_dim, "bf16", kv)
    for q, ctx, forms in (([1] * len(CTX), CTX, FORMS), ([1] * len(CTX) + [40], CTX + [70], MIXED), ([1] * 2, [2049, 3073], FORMS)):
        mk = lambda: make_batch(shape, q, ctx, seed=91, pool_rule=1.25, value_mult=0.5)
        ref, rk, rv = oracle.run_batch(W.to_cpu(mk()))
        for options in forms:
            print(f"[case] kv={kv} heads={heads} D={head_dim} rows={len(q)} {options}", flush=True)
            out, gk, gv = g.run_batch(mk(), options=options)
            again, _, _ = g.run_batch(mk(), options=options)
            assert gk.tobytes() == rk.tobytes() and gv.tobytes() == rv.tobytes()
            assert np.all(np.isfinite(out))
            worst = worst_of_rms(out, ref)
            print(f"       {worst:.4f} of the rms", flush=True)
            assert worst <= OF_RMS
            assert np.array_equal(out, again)
