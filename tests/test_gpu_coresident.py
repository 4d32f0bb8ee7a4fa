"""Decode rows next to resident prefill workgroups, two pages at a time: page counts per wave, head groups, scales."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from error_bar import OF_RMS, worst_of_rms
from workloads import AttnShape, make_batch

pytestmark = pytest.mark.gpu

CTX = [1, 15, 16, 17, 63, 64, 65, 79, 80, 81, 127, 128, 129, 130, 191, 192, 193, 255, 256, 257, 319, 321, 400, 511, 512, 513, 1000]


def gpu():
    import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("heads", [(16, 2), (10, 2), (2, 2), (7, 1), (8, 1), (18, 2), (32, 2)], ids=lambda h: f"{h[0]}q{h[1]}kv")
def test_decode_rows_next_to_resident_prefill_workgroups(kv, heads):
    """A wave of an item has 0 ... 16 pages, in pairs, with one or two left, the last of them full or not; whole rows
    and rows cut into items of 9 pages; at most eight heads per KV head (pairs) and more (single pages)."""
    b = make_batch(AttnShape(heads[0], heads[1], 128, "bf16", kv), [1] * len(CTX) + [40], CTX + [70], seed=81, pool_rule=1.25, value_mult=0.5)
    ref, rk, rv = oracle.run_batch(W.to_cpu(b))
    g = gpu()
    g.to_dev(b)
    for split, tiles in ((0, 2), (9, 2), (9, 3)):
        print(f"[case] kv={kv} heads={heads} split={split} tiles in flight={tiles}", flush=True)
        out, gk, gv = g.run_batch(b, options={"mixed_mode": 2, "prefill_resident_workgroups": 8, "decode_split_pages": split, "decode_prefetch_tiles": tiles})
        assert gk.tobytes() == rk.tobytes() and gv.tobytes() == rv.tobytes()
        assert np.all(np.isfinite(out))
        worst = worst_of_rms(out, ref)
        print(f"       {worst:.4f} of the rms", flush=True)
        assert worst <= OF_RMS


def test_decode_rows_next_to_tiles_with_a_negative_scale_and_infinite_values():
    """A negative K scale turns the order of the scores round; an infinite V of a page that its row sees reaches the
    output with its sign, whichever page of a pair it is in."""
    b = make_batch(AttnShape(8, 2, 128, "bf16", "fp8"), [1, 1, 1, 40], [300, 513, 64, 70], seed=82, pool_rule=1.25, value_mult=0.5)
    b.k_scale = torch.tensor([-0.02, 0.01])
    ref, _, _ = oracle.run_batch(W.to_cpu(b))
    out, _, _ = gpu().run_batch(b, options={"mixed_mode": 2, "prefill_resident_workgroups": 8})
    assert worst_of_rms(out[:3], ref[:3]) <= OF_RMS        # (the decode rows; the tiles expect positive scales)
    for page in (0, 4, 5, 18):                             # wave 0's first pair, wave 1's second page, the tail
        b = make_batch(AttnShape(8, 2, 128, "bf16", "bf16"), [1, 40], [300, 70], seed=83, pool_rule=1.25, value_mult=0.5)
        b.v_prefix[16 * page + 3, 1, 7] = float("inf")
        ref, _, _ = oracle.run_batch(W.to_cpu(b))
        out, _, _ = gpu().run_batch(b, options={"mixed_mode": 2, "prefill_resident_workgroups": 8})
        assert np.all(out[0, 4:, 7] == np.inf) and np.all(np.isinf(ref[0, 4:, 7]))
        keep = np.isfinite(ref)
        assert worst_of_rms(np.where(keep, out, 0), np.where(keep, ref, 0)) <= OF_RMS
