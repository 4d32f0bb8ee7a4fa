"""Sizes of the co-resident launch as planned: which decode rows are cut next to resident prefill workgroups."""
import pytest

import paper_2512_03416_amd as ts
from paper_2512_03416_amd import binding

# (query heads, cache, decode rows, chunk, prefix) of batches with a prefill workgroup on every CU, rows of 3000 tokens
# (188 pages, about 53 us next to tiles); microseconds of the chunk's tiles at 1.25 PFLOP/s
ROWS_NEXT_TO_TILES = [((32, "bf16", 12, 1024, 2300), 38, 2), ((32, "bf16", 12, 1500, 1500), 44, 2),
                      ((40, "bf16", 20, 2000, 1500), 82, 1), ((64, "fp8", 24, 1024, 1500), 54, 1)]


@pytest.mark.parametrize("batch,tiles_us,pieces", ROWS_NEXT_TO_TILES, ids=lambda x: str(x))
def test_rows_stay_whole_only_if_their_scan_ends_with_the_tiles(batch, tiles_us, pieces):
    heads, kv, rows, chunk, prefix = batch
    d = ts.Desc.make(heads, 8, 128, "bf16", kv, 1 << 16, 1 << 10)
    q, ctx = [1] * rows + [chunk], [3000] * rows + [prefix + chunk]
    info = ts.plan_describe(d, q, ctx)
    assert abs(4 * heads * 128 * (chunk * prefix + chunk * (chunk + 1) / 2) / 1.25e9 - tiles_us) < 1
    assert info.mixed_mode == 2 and info.n_decode_items == pieces * rows
    items = binding.plan_export(d, q, ctx, "decode")
    assert max(int(i[4] - i[3]) for i in items) * 0.28 <= tiles_us


# (cache, decode rows of 1024-8192 tokens, chunk, prefix) with 32/8 heads, resident workgroups: tiles of 0.5-0.8 of the scan's time
BETWEEN = [(("bf16", 128, 3968, 4096), range(256, 257)), (("bf16", 128, 3968, 3000), range(176, 209)), (("bf16", 128, 4600, 2000), range(176, 217)),
           (("bf16", 128, 3200, 4096), range(160, 217)), (("bf16", 128, 2400, 4096), range(120, 161)), (("fp8", 256, 3600, 3600), range(128, 169))]


@pytest.mark.parametrize("batch,workgroups", BETWEEN, ids=lambda x: str(x))
def test_tiles_of_more_than_half_the_scan_get_a_share_that_grows_with_them(batch, workgroups):
    """With the flat share they end late: 3968 tokens over 4096 615-629 us a pass with 152 workgroups, 533-548 with 224 or 256."""
    import numpy as np
    kv, rows, chunk, prefix = batch
    d = ts.Desc.make(32, 8, 128, "bf16", kv, 1 << 17, 1 << 10)
    ctx = np.random.default_rng(1).integers(1024, 8193, rows).tolist()
    info = ts.plan_describe(d, [1] * rows + [chunk], ctx + [prefix + chunk])
    assert info.mixed_mode == 2 and info.prefill_workgroups in workgroups, info.prefill_workgroups


# (query heads of 8 KV heads, cache, rows, shortest and longest, chunks, chunk, prefix): scans of less than 150 us
SHORT = [((32, "bf16", 50, 1500, 4800, 1, 3300, 1500), range(256, 257)), ((40, "bf16", 40, 1500, 4800, 1, 2600, 1000), range(256, 257)),
         ((64, "bf16", 24, 1500, 4800, 2, 1100, 300), range(176, 209)), ((128, "bf16", 30, 2000, 5000, 1, 1200, 800), range(256, 257)),
         ((32, "fp8", 60, 1500, 5000, 1, 2400, 1500), range(152, 193))]


@pytest.mark.parametrize("batch,workgroups", SHORT, ids=lambda x: str(x))
def test_short_scans_over_bf16_leave_the_tiles_more(batch, workgroups):
    """50 rows next to 3300 over 1500: 240 us a pass with 176 workgroups, 212 with 256; e4m3, 60 rows next to 2400 over 1500: 171
    with 176, 189 with 256."""
    import numpy as np
    heads, kv, rows, lo, hi, chunks, chunk, prefix = batch
    d = ts.Desc.make(heads, 8, 128, "bf16", kv, 1 << 17, 1 << 10)
    ctx = np.random.default_rng(2).integers(lo, hi + 1, rows).tolist()
    info = ts.plan_describe(d, [1] * rows + [chunk] * chunks, ctx + [prefix + chunk] * chunks)
    assert info.mixed_mode == 2 and info.prefill_workgroups in workgroups, info.prefill_workgroups


# 128 rows of 1024-8192 tokens next to a chunk: (query heads of 8 KV heads, cache, chunk, prefix), resident workgroups (with the plan of
# groups of up to eight heads: 256 for all but the second), items of at most 160 pages
WIDE_GROUPS = [((128, "bf16", 2048, 2048), range(176, 209), False), ((128, "bf16", 1024, 2048), range(96, 161), False),
               ((96, "bf16", 2500, 2000), range(176, 209), False), ((128, "fp8", 1500, 1500), range(120, 201), True),
               ((128, "bf16", 3072, 1000), range(256, 257), False)]


@pytest.mark.parametrize("batch,workgroups,cut", WIDE_GROUPS, ids=lambda x: str(x))
def test_groups_of_more_than_eight_heads_are_sized_by_their_own_measurements(batch, workgroups, cut):
    """Such a scan runs page by page and takes more from the tiles: not all CUs from 0.8 of its time on, and over a bf16 cache
    no cuts at 160 pages."""
    import numpy as np
    heads, kv, chunk, prefix = batch
    rows = np.random.default_rng(1).integers(1024, 8193, 128).tolist()
    d = ts.Desc.make(heads, 8, 128, "bf16", kv, 1 << 17, 1 << 10)
    info = ts.plan_describe(d, [1] * 128 + [chunk], rows + [prefix + chunk])
    assert info.mixed_mode == 2 and info.prefill_workgroups in workgroups and (info.split_pages <= 160) == cut


HARNESS = r"""
#include <cstdio>
#include <cstring>
#include <random>
#include "ts_internal.h"
using namespace ts;
template <typename T> static bool same(const std::vector<T>& a, const std::vector<T>& b)
{
    return a.size() == b.size() && (a.empty() || !memcmp(a.data(), b.data(), a.size() * sizeof(T)));
}
int main()
{
    std::mt19937 rng(11);
    auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    int mixed = 0, widened = 0;
    for (int it = 0; it < 1500; ++it) {
        ts_attn_desc d{};
        const int hkv[] = {1, 2, 4, 8};
        d.num_kv_heads = hkv[rng() % 4]; d.num_q_heads = d.num_kv_heads * pick(1, 16); d.head_dim = it % 4 ? 128 : 64;
        d.page_size = 16; d.num_pages = 1 << 20; d.max_pages_per_seq = 1 << 16;
        d.q_dtype = it % 7 ? TS_BF16 : TS_F32;
        d.kv_dtype = d.q_dtype == TS_F32 ? TS_F32 : it % 2 ? TS_BF16 : TS_FP8_E4M3;
        const int rows = pick(0, 200), chunks = pick(0, 6), most = 1 << pick(6, 13), len = 1 << pick(4, 12), before = 1 << pick(0, 13);
        std::vector<int32_t> q, c;
        for (int i = 0; i < rows; ++i) { q.push_back(1); c.push_back(pick(1, most)); }
        for (int i = 0; i < chunks; ++i) { q.push_back(pick(2, len)); c.push_back(q.back() + pick(0, before)); }
        if (q.empty()) continue;
        PlanOptions o, l;
        l.for_launch = true;
        Plan a, b;
        build_plan(d, q.data(), c.data(), (int)q.size(), o, &a);
        build_plan(d, q.data(), c.data(), (int)q.size(), l, &b);
        for (PfItem& t : b.pf) t.merge = 0;
        if (memcmp(&a.info, &b.info, sizeof a.info) || !same(a.dec, b.dec) || !same(a.dec_wg, b.dec_wg) || !same(a.cmb, b.cmb) || !same(a.pf, b.pf) ||
            !same(a.rt, b.rt) || !same(a.queue, b.queue) || !same(a.q_off, b.q_off) || !same(a.wide, b.wide)) {
            printf("batch %d: described %d workgroups, %d items, %lld partials, %lld widened; launched %d, %d, %lld, %lld\n", it, a.info.prefill_workgroups,
                   a.info.n_decode_items, (long long)a.info.partial_slots, (long long)a.info.widened_pages, b.info.prefill_workgroups,
                   b.info.n_decode_items, (long long)b.info.partial_slots, (long long)b.info.widened_pages);
            return 1;
        }
        mixed += b.info.mixed_mode == TS_MIXED_CORESIDENT;
        widened += b.info.widened_pages > 0;
    }
    printf("%d co-resident, %d widened\n", mixed, widened);
    return mixed > 50 && widened > 50 ? 0 : 2;
}
"""


def test_the_described_plan_is_the_launched_one(tmp_path):
    """Over random batches: the plan of a launch has the described counts and lists (but for the details that a launch
    adds: marks of tiles merged in the kernel, one record per run of fp32 tokens)."""
    import os
    import subprocess
    from paper_2512_03416_amd import build as B
    src = tmp_path / "plans.cpp"
    src.write_text(HARNESS)
    exe = str(tmp_path / "plans")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", B.CSRC, "-I", os.path.join(os.path.dirname(B.CSRC), "..", "include"), str(src),
                    os.path.join(B.CSRC, "ts_planner.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("head_dim,rows", [(128, 128), (64, 224)])
def test_the_default_places_are_those_of_the_kernels(head_dim, rows):
    """Rows stay whole up to as many workgroups as the GPU holds at once: four on a CU, seven with head dim 64."""
    d = ts.Desc.make(32, 8, head_dim, "bf16", "bf16", 1 << 16, 1 << 10)
    places = (4 if head_dim == 128 else 7) * 256
    for n in (rows - 1, rows, rows + 1):
        for ctx in ([1600] * n, [1600] * (n - 1) + [16000]):
            info = ts.plan_describe(d, [1] * n, ctx)
            stated = binding.plan_export(d, [1] * n, ctx, "decode", 0, places)
            assert (binding.plan_export(d, [1] * n, ctx, "decode") == stated).all() and info.n_decode_items == len(stated)
            assert n > rows or ctx[-1] > 1600 or len(stated) == n
