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
