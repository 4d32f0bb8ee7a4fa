"""fp32 decode rows of at most four heads per KV head (sixteen blocks of 4x4x1) against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from workloads import AttnShape, make_batch

pytestmark = pytest.mark.gpu

CTX = [1, 2, 15, 16, 17, 63, 64, 65, 80, 81, 127, 128, 129, 255, 257, 700]


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("heads", [(2, 2), (4, 2), (6, 2), (8, 2), (10, 2)], ids=lambda h: f"{h[0]}q{h[1]}kv")
def test_fp32_decode_rows_alone_and_next_to_a_chunk(heads, head_dim):
    """Rows whose waves have no page, one, several, the last full or not, whole and cut; five heads per KV head take the
    sixteen-column form."""
    import gpu_harness as g
    for q, ctx in (([1] * len(CTX), CTX), ([1] * len(CTX) + [21], CTX + [50]), ([1, 1], [3000, 2999])):
        b = make_batch(AttnShape(heads[0], heads[1], head_dim, "f32", "f32"), q, ctx, seed=91, pool_rule=1.25, value_mult=0.5)
        ref, rk, rv = oracle.run_batch(W.to_cpu(b))
        print(f"[case] heads={heads} D={head_dim} rows={len(q)}", flush=True)
        out, gk, gv = g.run_batch(b)
        assert gk.tobytes() == rk.tobytes() and gv.tobytes() == rv.tobytes()
        assert float(np.max(np.abs(out - ref))) <= 1e-5
        again, _, _ = g.run_batch(b)
        assert np.array_equal(out, again)


def test_fp32_decode_row_with_an_infinite_value():
    """An infinite V of a cached token reaches the output of its head group; an unwritten slot never does."""
    import gpu_harness as g
    b = make_batch(AttnShape(4, 1, 64, "f32", "f32"), [1], [200], seed=92, pool_rule=1.25, value_mult=0.5)
    b.v_prefix[37, 0, 5] = float("-inf")
    ref, _, _ = oracle.run_batch(W.to_cpu(b))
    out, _, _ = g.run_batch(b)
    assert np.all(out[0, :, 5] == -np.inf) and np.array_equal(np.isfinite(out), np.isfinite(ref))
    keep = np.isfinite(ref)
    assert float(np.max(np.abs(out[keep] - ref[keep]))) <= 1e-5
