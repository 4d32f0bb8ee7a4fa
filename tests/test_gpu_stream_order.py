"""Co-resident passes end on two streams: the tiles on the caller's, the decode rows and their merge on the context's own.  What
comes after one -- a pass on another stream, a wait for the end -- has to come after both."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from error_bar import OF_RMS, worst_of_rms
from workloads import AttnShape, make_batch

pytestmark = pytest.mark.gpu

ROWS, CTX = 256, 3000                                      # a scan of about 100 us next to a chunk that takes a fraction of that
OPTIONS = {"prefill_resident_workgroups": 8, "decode_split_pages": 64}


def batch(kv, seed):
    """Every row is cut, and there are more items than the GPU holds at once, so work lists and partials are read to the end."""
    rng = np.random.default_rng(seed)
    ctx = sorted(rng.integers(CTX // 2, CTX, ROWS).tolist(), reverse=bool(seed % 2)) + [70]
    return make_batch(AttnShape(16, 4, 128, "bf16", kv), [1] * ROWS + [40], ctx, seed=seed, num_pages=ROWS * CTX // 16 + 100, value_mult=0.5)


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_a_pass_on_another_stream_follows_both_ends_of_a_co_resident_one(kv):
    """Two batches of one context in turn on two streams, without a host synchronisation: the second pass rewrites the work
    lists and the partial results of the first, whose tiles ended long before its scan.  e4m3: the chunk's few pages
    are copied, so the decode grid starts behind the copy."""
    import gpu_harness as g
    import paper_2512_03416_amd as ts
    two = [batch(kv, 1), batch(kv, 2)]
    refs = [oracle.run_batch(W.to_cpu(b))[0] for b in two]
    two = [g.to_dev(b) for b in two]
    width = max(b.max_pages_per_seq for b in two)
    desc = ts.Desc.make(16, 4, 128, "bf16", kv, two[0].num_pages, width)
    info = ts.plan_describe(desc, two[0].q_lens, two[0].ctx_lens, 64)
    assert info.n_combine_rows == ROWS and info.n_decode_items * 4 > 2048 and info.widened_pages == (5 if kv == "fp8" else 0)
    ctx = ts.Context(desc)
    for name, value in OPTIONS.items():
        ctx.set_option(name, value)
    calls = []
    for b in two:
        kc, vc = g.new_caches(b)
        table = np.full((b.num_seqs, width), -1, np.int32)
        table[:, :b.block_table.shape[1]] = b.block_table
        bt = torch.from_numpy(table).cuda()
        ctx.kv_append(b.k_prefix, b.v_prefix, kc, vc, b.k_scale, b.v_scale, bt, b.prefix_lens, b.prefix_lens)
        calls.append((b.q, b.k_new, b.v_new, kc, vc, b.k_scale, b.v_scale, bt, b.q_lens, b.ctx_lens, b.sm_scale, torch.zeros_like(b.q)))
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(6):                                     # one by one, until the probe of the side stream is settled
        for c in calls:
            ctx.mixed_paged_attention(*c, stream=s1)
            torch.cuda.synchronize()
    alone = [c[-1].clone() for c in calls]
    for out, ref in zip(alone, refs):
        worst = worst_of_rms(out.double().cpu().numpy(), ref)
        print(f"[case] kv={kv} {worst:.4f} of the rms", flush=True)
        assert worst <= OF_RMS
    for order in ((0, 1), (1, 0), (0, 1, 0, 1, 0, 1)):
        for c in calls:
            c[-1].zero_()
        torch.cuda.synchronize()
        for k, i in enumerate(order):
            ctx.mixed_paged_attention(*calls[i], stream=(s1, s2)[k % 2])
        torch.cuda.synchronize()
        for c, out in zip(calls, alone):
            assert torch.equal(c[-1], out), (kv, order)
    # an append on another stream: its work list shares the buffer
    for c in calls:
        c[-1].zero_()
    torch.cuda.synchronize()
    ctx.mixed_paged_attention(*calls[0], stream=s1)
    many = [1] * (ROWS + 1)
    b = two[1]
    ctx.kv_append(b.k_new[:ROWS + 1], b.v_new[:ROWS + 1], calls[1][3], calls[1][4], b.k_scale, b.v_scale, calls[1][7], many, many, stream=s2)
    torch.cuda.synchronize()
    assert torch.equal(calls[0][-1], alone[0])
    # the counters' wait is for the end of the scan as well: a stream that is ordered behind nothing finds the rows written
    s3 = torch.cuda.Stream()
    for _ in range(3):
        calls[0][-1].zero_()
        torch.cuda.synchronize()
        ctx.mixed_paged_attention(*calls[0], stream=s1)
        ctx.token_velocity(sync=True)
        with torch.cuda.stream(s3):
            seen = calls[0][-1].cpu()
        torch.cuda.synchronize()
        assert torch.equal(seen, alone[0].cpu())
    ctx.close()


@pytest.mark.parametrize("other", [False, True], ids=["same stream", "other stream"])
@pytest.mark.parametrize("form", ["fused", "one launch per class", "co-resident", "co-resident, copied pages", "fp32"])
def test_captured_passes_between_eager_ones(form, other):
    """Events ride on the kernels of eager passes and are recorded in captured ones: a pass captured behind eager ones of the
    same context, on their stream or another, and replayed with eager passes in between, gives the same bytes each time."""
    import gpu_harness as g
    import paper_2512_03416_amd as ts
    q, c, kv, dtype, options = {"fused": ([1, 1], [500, 900], "bf16", "bf16", {}),
                                "one launch per class": ([1, 1, 40], [500, 900, 70], "bf16", "bf16", {}),
                                "co-resident": ([1] * 40 + [40], [2000] * 40 + [70], "bf16", "bf16", {"prefill_resident_workgroups": 8}),
                                "co-resident, copied pages": ([1] * 40 + [40], [2000] * 40 + [70], "fp8", "bf16", {"prefill_resident_workgroups": 8}),
                                "fp32": ([1] * 4 + [40], [200] * 4 + [70], "f32", "f32", {})}[form]
    b = make_batch(AttnShape(16, 4, 128, dtype, kv), q, c, seed=3, pool_rule=1.2, value_mult=0.5)
    ref = oracle.run_batch(W.to_cpu(b))[0]
    b = g.to_dev(b)
    print(f"[case] captured: {form}, other stream {other}", flush=True)
    ctx = ts.Context(g.make_desc(b))
    for name, value in options.items():
        ctx.set_option(name, value)
    ctx.reserve(b.total_q, b.num_seqs, sum(-(-n // 16) for n in c))
    kc, vc = g.new_caches(b)
    bt = torch.from_numpy(b.block_table).cuda()
    ctx.kv_append(b.k_prefix, b.v_prefix, kc, vc, b.k_scale, b.v_scale, bt, b.prefix_lens, b.prefix_lens)
    out = torch.zeros_like(b.q)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()

    def call(stream):
        ctx.mixed_paged_attention(b.q, b.k_new, b.v_new, kc, vc, b.k_scale, b.v_scale, bt, b.q_lens, b.ctx_lens, b.sm_scale, out, stream=stream)
    for _ in range(2):
        call(s1)
        torch.cuda.synchronize()
    want = out.clone()
    assert worst_of_rms(want.double().cpu().numpy(), ref) <= OF_RMS
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s2 if other else s1, capture_error_mode="relaxed"):
        call(s2 if other else s1)
    for _ in range(3):
        for again in (graph.replay, lambda: call(s1)):
            out.zero_()
            torch.cuda.synchronize()
            again()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
    ctx.close()
