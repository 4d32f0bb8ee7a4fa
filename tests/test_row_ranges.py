"""How the tiles of the generic kernel are cut along the pages: ranges of a fair share of the GPU's places (two
workgroups on each of 256 CUs); where chunks have two fifths of all pages or more, twice that for decode rows, and none at all while
no tile is longer than twice the share."""
import pytest

import paper_2512_03416_amd as ts
from paper_2512_03416_amd import binding

HEADS = (32, 8)                                            # tiles of four tokens

BATCHES = {                                                # (query lengths, prefixes)
    "a short chunk over a long prefix": ([64], [16384]),
    "chunk tiles of nearly a share": ([240], [500]),
    "chunk tiles of twice a share": ([150], [1500]),
    "a ragged last tile": ([150, 5], [1000, 9000]),
    "decode rows alone": ([1] * 32, [500 + 50 * i for i in range(32)]),
    "both": ([1] * 30 + [300, 100, 257], [500 + 150 * i for i in range(30)] + [0, 500, 300]),
    "both, hardly any chunk": ([1] * 43 + [37], [220 + 40 * i for i in range(43)] + [200]),
    "both, none longer than twice a share": ([1] * 20 + [100, 150], [360 + 4 * i for i in range(20)] + [400, 700]),
    "both, few pages": ([1] * 4 + [200, 300], [100, 40, 600, 333, 0, 100]),
    "both, a long prefix": ([1] * 8 + [100], [1000 + 125 * i for i in range(8)] + [4000]),
}


@pytest.mark.parametrize("batch", list(BATCHES))
def test_ranges_of_generic_row_tiles(batch):
    q, prefix = BATCHES[batch]
    d = ts.Desc.make(HEADS[0], HEADS[1], 128, "f32", "f32", 1 << 16, 1 << 11)
    tiles, row = [], 0                                     # (first row, tokens, pages, decode row)
    for n, p in zip(q, prefix):
        for i in range(0, n, 4):
            cnt = min(4, n - i)
            tiles.append((row + i, cnt, (p + i + cnt - 1) // 16 + 1, n == 1))
        row += n
    share = max(16, -(-sum(t[2] for t in tiles) * HEADS[1] // 512))
    chunk_share = sum(t[2] for t in tiles if not t[3]) / sum(t[2] for t in tiles)
    want = {}
    for first, cnt, pages, dec in tiles:
        most = 2 * share if share >= 32 and dec and chunk_share >= 0.4 else share
        if share >= 32 and chunk_share >= 0.4 and max(t[2] for t in tiles) <= 2 * share:
            most = pages
        n = -(-pages // most)
        n = -(-pages // (-(-pages // n)))
        if n > 1:
            want.update({first + i: n for i in range(cnt)})
    ctx = [a + b for a, b in zip(q, prefix)]
    got = {int(r): int(n) for r, _, n, _ in binding.plan_export(d, q, ctx, "combine")}
    assert got == want
    assert ts.plan_describe(d, q, ctx).partial_slots == sum(want.values())
    if batch == "a short chunk over a long prefix":        # every place of the GPU gets a workgroup
        assert sum(want.values()) // 4 * HEADS[1] >= 512
    assert bool(want) == (batch not in ("chunk tiles of nearly a share", "chunk tiles of twice a share", "both, none longer than twice a share"))
