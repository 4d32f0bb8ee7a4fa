// Host work planner (step a0): turns the per-sequence lengths of one iteration's batch into the
// device work lists.  Pure host code, no GPU calls.
//
// The batch is the one a Convertible Decoder forms each iteration: its decode batch plus the
// prefill chunk(s) it absorbed, bounded by the profiled chunk size (paper Sec. 4.4).  Decode rows
// are cut into split-K items over the sequence's page list so that an HBM-bound scan is spread
// over all CUs; prefill chunks are cut into causal query tiles.  Items are ordered longest first
// so that the hardware dispatcher, which hands out workgroups in order, balances the tail.
#include <algorithm>
#include <array>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <functional>
#include <utility>

#include "ts_internal.h"

namespace ts {

bool desc_uses_mfma(const ts_attn_desc& d)
{
    return d.q_dtype == TS_BF16 && d.head_dim == 128 &&
           (d.kv_dtype == TS_BF16 || d.kv_dtype == TS_FP8_E4M3);
}

bool desc_uses_mfma_decode(const ts_attn_desc& d)
{
    return d.q_dtype == TS_BF16 && (d.head_dim == 128 || d.head_dim == 64) &&
           (d.kv_dtype == TS_BF16 || d.kv_dtype == TS_FP8_E4M3);
}

bool desc_uses_mfma_tiles(const ts_attn_desc& d)
{
    return desc_uses_mfma_decode(d);
}

int32_t prefill_tile_tokens(const ts_attn_desc& d)
{
    int G = d.num_q_heads / d.num_kv_heads;
    return 256 / G;     // 256 query rows (token, head-in-group) per tile
}

static int check_desc_impl(const ts_attn_desc* d, std::string* err)
{
    auto fail = [&](int code, const char* msg) { if (err) *err = msg; return code; };
    if (!d) return fail(TS_ERR_INVALID_ARG, "descriptor is NULL");
    if (d->page_size != kPage) return fail(TS_ERR_INVALID_ARG, "page_size must be 16");
    if (d->num_q_heads <= 0 || d->num_kv_heads <= 0 || d->num_q_heads % d->num_kv_heads)
        return fail(TS_ERR_INVALID_ARG, "num_q_heads must be a positive multiple of num_kv_heads");
    if (d->num_pages <= 0 || d->max_pages_per_seq <= 0)
        return fail(TS_ERR_INVALID_ARG, "num_pages and max_pages_per_seq must be positive");
    if (d->num_pages * (int64_t)d->num_kv_heads >= (int64_t)1 << 31)
        return fail(TS_ERR_INVALID_ARG, "num_pages * num_kv_heads must stay below 2^31");
    if (d->head_dim != 64 && d->head_dim != 128)
        return fail(TS_ERR_UNSUPPORTED, "head_dim must be 64 or 128");
    if (d->num_q_heads / d->num_kv_heads > 16)
        return fail(TS_ERR_UNSUPPORTED, "more than 16 query heads per KV head");
    bool ok = (d->q_dtype == TS_F32 && d->kv_dtype == TS_F32) ||
              (d->q_dtype == TS_BF16 && d->kv_dtype == TS_BF16) ||
              (d->q_dtype == TS_BF16 && d->kv_dtype == TS_FP8_E4M3);
    if (!ok) {
        bool known = d->q_dtype >= TS_F32 && d->q_dtype <= TS_FP8_E4M3 && d->kv_dtype >= TS_F32 &&
                     d->kv_dtype <= TS_FP8_E4M3;
        return fail(known ? TS_ERR_UNSUPPORTED : TS_ERR_INVALID_ARG,
                    "dtype pair must be (f32,f32), (bf16,bf16) or (bf16,fp8_e4m3)");
    }
    return TS_OK;
}

int validate_batch(const ts_attn_desc& d, const int32_t* q_lens, const int32_t* ctx_lens,
                   int num_seqs, std::string* err)
{
    char buf[160];
    if (num_seqs < 0) { *err = "num_seqs is negative"; return TS_ERR_INVALID_ARG; }
    if (num_seqs > 0 && (!q_lens || !ctx_lens)) {
        *err = "q_lens / ctx_lens is NULL";
        return TS_ERR_INVALID_ARG;
    }
    int64_t total = 0;
    for (int s = 0; s < num_seqs; ++s) {
        if (q_lens[s] < 0 || ctx_lens[s] < q_lens[s]) {
            snprintf(buf, sizeof buf, "sequence %d: q_len %d, ctx_len %d (need 0 <= q_len <= ctx_len)",
                     s, q_lens[s], ctx_lens[s]);
            *err = buf;
            return TS_ERR_INVALID_ARG;
        }
        if ((int64_t)ctx_lens[s] > (int64_t)kPage * d.max_pages_per_seq) {
            snprintf(buf, sizeof buf, "sequence %d: ctx_len %d exceeds 16 * max_pages_per_seq (%d)", s,
                     ctx_lens[s], d.max_pages_per_seq);
            *err = buf;
            return TS_ERR_INVALID_ARG;
        }
        total += q_lens[s];
    }
    if (total >= ((int64_t)1 << 31) / std::max(1, d.num_q_heads * d.head_dim / 64)) {
        *err = "batch has too many query tokens";
        return TS_ERR_INVALID_ARG;
    }
    return TS_OK;
}

// How the decode rows are cut.  A row that fits one item is finished by its workgroup without any partial result
// in HBM.  Two facts decide the rest (measured): the memory system serves the CUs alike, so that what counts is the
// pages per CU, and a launch of one item per CU and a bit (a few CUs with two) takes nearly twice as long as one of
// exactly one per CU; and every item costs its start (page ids, queries, first tiles: 2-3 us, hidden only by other
// workgroups of the CU) and every cut its partial results and their merge.  So, for a launch of decode items alone:
//   1. rows that give every CU a workgroup and come out even over the CUs stay whole (rows_stay_whole);
//   2. else long batches are dealt out evenly: each workgroup gets the same number of pages, whatever rows they
//      belong to (deal_decode_evenly);
//   3. else (less than a workgroup per CU): pieces of one length, the shortest with which the items do not
//      outnumber the CUs, and at least 32 pages (auto_split_pages).  8 rows of 1500 tokens in pieces of 32 pages
//      take 17.3 us a pass, in pieces of 28 (a few items more than CUs) 20.5; 16 rows of 500-3000 tokens 28.1 us
//      in 28 items per KV head, 36.2 us in pieces of 32 pages (64 items);
//   4. batches whose rows outnumber the workgroup slots (those of decode_kernel_lean, see rows_stay_whole): a row is cut when it exceeds 5/4 of a workgroup slot's
//      fair share, and the dispatcher balances the items, longest first (180 rows of 600-5700 tokens: 382 us
//      against 390 cut at the fair share itself; with a heavy tail, 600-25 700 tokens and e4m3: 290, at 3/2: 298,
//      uncut: 382).
// In a mixed batch launched with resident workgroups (co-resident launch or one persistent kernel: a CU that
// holds a resident workgroup has room for one decode workgroup, a quarter of the stand-alone slots), 3 does not
// apply and the fair share is that of the slots actually there: measured on the burst configuration,
// 706 -> 692 us and no combine launch.
// Rates the two kinds of work reach on their own (decode scan: bytes per microsecond; prefill tiles: flop per
// microsecond, all CUs).
constexpr double kDecBytePerUs = 6.2e6;
constexpr double kPfFlopPerUs = 1.25e9;
// Co-resident launch: the CUs that get a resident prefill workgroup, from the ratio r of the two times (prefill to decode).
// All of them where the tiles would take about as long as the scan or longer (r >= kPfAllRatio; passes with a scan of less
// than kPfAllUs: r >= kPfAllRatioShort, over an e4m3 cache kPfAllRatioShort8): a CU without one takes four decode workgroups, each of them then four times as slow as
// the ones that share a CU with tiles, and the longest rows end late there (248 workgroups instead of 256: 568 us for 510
// in the first example below).  Else the share kPfShare0 + kPfShare1 * r; beside a bf16 scan of kPfAllUs or more
// at least kPfSteep0 + kPfSteep1 * r, which is the larger from r = 0.45 on.  Measured over 60 mixed batches, every multiple of 16
// workgroups: with too few the tiles end late (the time rises steeply), with a few too many the scan does.
// 128 rows of 1024-8192 tokens next to 4096 over 4096 (r = 0.83): 508 us with 256, 576 with 192; 4 chunks of 2048 (r = 0.97): 585 and
// 640; r > 1.7 always 256.  Over 49 of them with r = 0.07 ... 0.96 this is within 1.4 % of the best number on average (6.7 % at
// most).  With the flat share alone bf16 batches between r = 0.5 and 0.8 get too few: next to 3968 over 4096 (r = 0.79) 629 us a
// pass with 152 workgroups, 533 with 256; 3968 over 3000 (0.65) 557 with 144, 522 with 192; 4600 over 2000 (0.65) 549 and 513; 8 chunks of
// 700-1100 (0.59) 560 with 144, 533 with 176.  Next to an e4m3 scan, which takes more of the SIMDs per byte, it is enough: 256 rows, 3600 over
// 3600 (0.65) 621 with 144, 630 with 192.
// Short scans over bf16: at least kPfShort0 + kPfShort1 * r (the larger from r = 0.71 on), 16 batches with r = 0.51 ... 1.7, within 0.9 % of
// the best on average.  The line of the e4m3 ones, 1.4, held for both before: 50 rows of 1500-4800 next to 3300 over 1500 (r = 1.32) 240 us with
// 176 workgroups, 212 with 256; 40/8 heads, 40 rows next to 2600 over 1000 (1.18) 184 and 166; 24 rows next to 2 chunks of 1100 (64/8 heads,
// 0.96) 123 with 160, 116 with 192.  e4m3: 60 rows next to 2400 over 1500 (1.32) 171 with 176, 189 with 256; 64/8 heads, 1700 over 1000
// (1.33) 172 and 182.
constexpr double kPfShare0 = 0.46, kPfShare1 = 0.16, kPfSteep0 = 0.1, kPfSteep1 = 0.96, kPfShort0 = 0.12, kPfShort1 = 0.64;
constexpr double kStageUs = 1.5;                           // a tile's 64 keys
constexpr double kPfAllRatio = 0.75, kPfAllUs = 150.0, kPfAllRatioShort = 1.1, kPfAllRatioShort8 = 1.4;
// With more than eight query heads per KV head the scan takes its pages one by one (decode_kernel_lean_merging) and costs the tiles
// more where they share a CU: all CUs from kPfAllRatioWide on; below, over bf16 caches, the share grows faster with r.  Scans of kPfAllUs
// and more next to one chunk, 128 rows of 1024-8192 tokens, us a pass: 128/8 heads, 2048 over 2048 (r = 0.83) 602-610 with 256 workgroups,
// 597 with 192 and 633 with 160, 3072 over 1000 (1.02) 645, 688 and 737; 96/8 heads, 2500 over 2000 (0.80) 619, 581 and 620; e4m3, 128/8
// heads, 1500 over 1500 (0.89) 443, 399 and 404, 390 with 128; e4m3, 256 rows next to 2500 over 1500 (0.91) 734, 723 and 723.
constexpr double kPfAllRatioWide = 1.0, kPfShare0Wide = 0.25, kPfShare1Wide = 0.6;
// A mixed batch is launched class by class when either class is estimated below this many microseconds: running
// side by side hides about 40 % of the shorter class, and the fork and join of the co-resident launch cost
// 10-15 us.  Measured: 128 decode rows (395 us) next to a chunk of 128 / 896 tokens without prefix (estimates
// 0.1 / 5 us): 0.410 / 0.425 ms class by class against 0.423 / 0.432 ms; next to 384 tokens over a prefix of 4096
// (22 us): 0.450 against 0.429 ms; 16 decode rows of 2500 tokens (26 us) next to 256 tokens over 4096 (14 us):
// 85 against 89 us; 8 rows of 1500 tokens (8 us) next to 1024 tokens over 2048 (34 us): 85 against 100 us.
constexpr double kCoresidentMinUs = 20.0;

constexpr int64_t kMinSplitPages = 32;
// Co-resident launch.  A CU with a resident prefill workgroup serves its one decode workgroup faster than a CU without
// one serves each of its four, so items of a workgroup's fair share do not end together.  Where the rows are few (less
// than one and a half times the slots of the whole GPU), items of at most kCoItemPages pages let the dispatch even it out: 64
// rows of 2000-16 000 tokens next to 16 chunks of 300-1024 499 -> 470 us, 16 rows of 8000-64 000 (e4m3) next to 8 chunks
// of 100-300 386 -> 331, 3072 tokens over 2048 next to 128 rows of 1024-8192 514 -> 468; with more rows the partial results
// cost more than it gains (256 rows of 1024-8192 tokens, e4m3, 474 -> 517; 512 of 512-4096 786 -> 818), and so they do for groups of
// more than eight heads over a bf16 cache (128 rows of 1024-8192, 128/8 heads, next to 1024 over 2048 471 -> 494, next to 512 over
// 4096 452 -> 478; 96/8 heads, 1500 over 2000, 478 -> 503; e4m3, 1500 over 1500, 442 -> 407).  With a prefill
// workgroup on every CU rows of up to kWholePages pages stay whole if their scan, kCoPageUs a page next to tiles, ends within the
// tiles' time: 20 rows of 3000 tokens (188 pages, 53 us) next to 2000 over 1500 (tiles 82 us) 131.0 us a pass, in pieces of 72-160 pages
// 138; 24 e4m3 rows of 3000 next to 1024 over 1500 (54 us) 98 and 101; 24 rows of 300-3000 next to 2024 over 1000 (67 us) 109.6 and 111;
// but 12 of 3000 next to 1024 over 2300 (38 us) 100.8 whole and 86.3 in two, 16 of 1500-3000 next to 1500 over 1000 (40/8 heads, 43
// us) 94.4 and 86.5, 12 of 3000 next to 1500 over 1500 (44 us) 94.2 and 90.0.
constexpr int64_t kCoItemPages = 160, kWholePages = 192;
constexpr double kCoPageUs = 0.28;

static int32_t auto_split_pages(const Plan& p, int num_seqs, int64_t decode_tiles, int64_t decode_pages, int Hkv,
                                int32_t wg_slots, int32_t n_cu, bool filled_by_prefill, int32_t pf_wgs, double t_pf,
                                bool wide_bf16)
{
    // (next to a resident prefill workgroup a CU has room for one decode workgroup; the CUs without one hold
    // their usual share of the stand-alone slots)
    int64_t slots = std::max<int32_t>(1, filled_by_prefill ? n_cu : wg_slots);
    if (filled_by_prefill && pf_wgs > 0 && pf_wgs < n_cu)
        slots = pf_wgs + (int64_t)(n_cu - pf_wgs) * std::max(1, wg_slots / n_cu);
    int64_t L = std::max<int64_t>(kMinSplitPages, (decode_tiles + slots - 1) / slots);
    if (pf_wgs >= n_cu) L = std::max(L, std::min(kWholePages, (int64_t)(t_pf / kCoPageUs)));
    else if (pf_wgs > 0 && !wide_bf16 && 2 * p.info.decode_tokens * Hkv < 3 * wg_slots) L = std::min(L, kCoItemPages);
    if (!filled_by_prefill && p.info.decode_tokens * Hkv <= n_cu && decode_pages > 0) {
        const int64_t want_items = std::max<int64_t>(1, n_cu / Hkv);   // per KV head
        int64_t fit = std::max<int64_t>(kMinSplitPages, (decode_pages + want_items - 1) / want_items);
        auto items = [&] {
            int64_t n = 0;
            for (int s = 0; s < num_seqs; ++s)
                if (p.seqs[s].q_len == 1) n += ((p.seqs[s].ctx_len + kPage - 1) / kPage + fit - 1) / fit;
            return n;
        };
        for (int tries = 0; tries < 64 && items() > want_items; ++tries) fit += std::max<int64_t>(1, fit / 16);
        L = fit;
    }
    return (int32_t)std::min<int64_t>(L, 1 << 20);
}

// Generic row tiles longer than a fair share of the workgroups that the GPU holds at once (two of four waves per
// CU) are cut along the pages into ranges of at most that share; a range has at least 16 pages (four per wave:
// shorter ones spend longer starting up and merging than multiplying).
// From shares of kRowTileLongPages pages on (fewer: 4 rows and 2 chunks 33.8 -> 35.2 with longer ones):
//   - ranges of decode rows next to chunk tiles, which the matrix instruction bounds, are twice as long: half the workgroups
//     keep enough of the scan on the way, and the chunk tiles, cut as ever, find more places from the start (32/8 heads of 128, 30
//     rows of 500-2000 tokens and 3 chunks of 100-300 91.5 -> 85.9 us a pass, 16 rows of 1000-2048 and a chunk of 231 over 1000
//     79.0 -> 72.2; rows without chunks are slower, 67.5 -> 74.0).  Where the chunk tiles have kRowChunkShare of all pages or more, over
//     150 random mixes: ranges twice as long take 0.92 of the time there on average, 1.01 at shares of 0.1-0.4 and 1.05 below
//     (43 rows of 220-1900 next to 37 tokens over 200 75.7 and 69.4 us).  Groups of more than four heads, whose rows the matrix
//     instruction bounds too, from kRowChunkShareWide on: 0.97 of the time between the two lines (64/8 heads, 24 rows of 1106-1501 next
//     to 80 over 400 52.1 and 61.6);
//   - from the same lines on all tiles stay whole where none is longer than twice the share (they give every CU a workgroup then): cut,
//     their ranges would be more than the places, one short round behind the other, and a merge (one chunk of 240 tokens over
//     500 46.2 -> 32.5, of 150 over 1000 47.6 -> 44.1, over 1500 58.0 -> 58.9; 64/8 heads, 9 rows of 458-618 next to 2 chunks of 29-53
//     over 615-653 46.4 -> 33.0).  Longer chunk tiles are cut at the share (64 tokens over 16384: 143 us; at twice the share 153).
constexpr int kRowTileMinPages = 16, kRowTileWgsPerCu = 2, kRowTileLongPages = 32;
constexpr double kRowChunkShare = 0.4, kRowChunkShareWide = 0.15;

static int32_t row_tile_tokens(const ts_attn_desc& d) { return 16 / (d.num_q_heads / d.num_kv_heads); }

// At most S / Hkv tiles exceed a fair share of S slots, and they are cut into at most 2 S / Hkv ranges; and no token
// has more partial results than its pages make ranges.
int64_t row_tile_slots_bound(const ts_attn_desc& d, int32_t n_cu, int64_t max_tokens, int64_t max_ctx_pages)
{
    return std::min(2 * (int64_t)row_tile_tokens(d) * (kRowTileWgsPerCu * (int64_t)n_cu / d.num_kv_heads + 1),
                    max_tokens * (max_ctx_pages / kRowTileMinPages + 1));
}

static int32_t row_tile_pages(const Plan& p, const RowTile& t)
{
    const int32_t cut = t.n_tok_cut >> 8;
    return cut ? p.rtcut[cut - 1].page_end - p.rtcut[cut - 1].page_begin : (t.pos0 + t.n_tok_cut - 1) / kPage + 1;
}

static int32_t cut_row_tiles(Plan& p, int G, int Hkv, const PlanOptions& opt, int32_t part)
{
    const int64_t slots = kRowTileWgsPerCu * (int64_t)std::max(1, opt.n_cu);
    if (opt.row_cut_few_only && (int64_t)p.rt.size() * Hkv >= slots) return part;
    auto decode_row = [&](const RowTile& t) { return p.seqs[t.seq].q_len == 1; };
    int64_t pages = 0, chunk_pages = 0;
    for (const RowTile& t : p.rt) {
        pages += row_tile_pages(p, t);
        if (!decode_row(t)) chunk_pages += row_tile_pages(p, t);
    }
    const int32_t L = (int32_t)std::max<int64_t>(kRowTileMinPages, (pages * Hkv + slots - 1) / slots);
    const bool longer = L >= kRowTileLongPages && chunk_pages >= (G <= 4 ? kRowChunkShare : kRowChunkShareWide) * pages;
    if (longer && std::all_of(p.rt.begin(), p.rt.end(), [&](const RowTile& t) { return row_tile_pages(p, t) <= 2 * L; })) return part;
    const int32_t L_dec = longer ? 2 * L : L;
    auto cuts = [&](const RowTile& t) {
        const int32_t most = decode_row(t) ? L_dec : L;
        return (row_tile_pages(p, t) + most - 1) / most;
    };
    int64_t need = part;
    for (const RowTile& t : p.rt)
        if (cuts(t) > 1) need += (int64_t)cuts(t) * t.n_tok_cut;
    if (need > opt.part_slots) return part;
    std::vector<RowTile> whole;
    whole.swap(p.rt);
    for (const RowTile& t : whole) {
        const int32_t n_pages = row_tile_pages(p, t), want = cuts(t), per = (n_pages + want - 1) / want, n_split = (n_pages + per - 1) / per;
        if (n_split == 1) { p.rt.push_back(t); continue; }
        for (int32_t i = 0; i < t.n_tok_cut; ++i) p.cmb.push_back(CmbItem{t.row0 + i, part + i * n_split, n_split, 0});
        for (int32_t k = 0; k < n_split; ++k) {
            p.rtcut.push_back(RowCut{k * per, std::min(n_pages, (k + 1) * per), part + k, n_split});
            p.rt.push_back(RowTile{t.seq, t.row0, t.pos0, t.n_tok_cut | (int32_t)(p.rtcut.size() << 8)});
        }
        part += t.n_tok_cut * n_split;
    }
    return part;
}

// Decode items dealt out evenly: every workgroup gets the same number of pages, whatever rows they belong to; one
// workgroup per CU (two where a tile is only 2 KB, head dim 64 and e4m3; twice as many where the rows are many, so that
// a workgroup has not more than two or three).  Its waves have three KV tiles in flight (two where a tile is 2 KB), except
// in passes whose lists are kernel arguments -- of the batches below the first three --: decode_kernel_fused has two.
// Measured against pieces of one length: 3 rows of 30-131 Ki tokens (64/8 heads, e4m3) 95 us for 119-123, 48 rows of
// 200-6000 tokens (head dim 64) 57.6 for 61.9, 20 rows of 500-8000 tokens 62 for 74, 100 rows of 1600-5700 tokens
// (e4m3) 142 for 150; shares below about 80 pages lose to rule 3 (16 rows of 500-4000 tokens, e4m3, 68 pages each:
// 24.6 us against 23.8).
constexpr int64_t kItemPages = 4;                          // pages that the start and the merge of an item are worth
constexpr int64_t kMinEvenShare = 80;
constexpr int32_t kMaxItemsPerWg = 48;                     // (the workgroup counts its arrivals with one wave: at most 64)

static bool deal_decode_evenly(Plan& p, int num_seqs, int64_t pages, const ts_attn_desc& d, const PlanOptions& opt, int32_t* part)
{
    const int64_t Hkv = d.num_kv_heads, per_cu = std::max<int64_t>(1, opt.n_cu / Hkv), rows = p.info.decode_tokens;
    const int64_t total = pages + rows * kItemPages;
    const bool small_tile = d.head_dim == 64 && d.kv_dtype == TS_FP8_E4M3;
    int64_t k = small_tile ? 2 : 1;
    if (rows >= 2 * k * per_cu) k *= 2;
    const int64_t W = k * per_cu;                          // workgroups per KV head
    if (rows >= 2 * W || total < W * kMinEvenShare || W + rows > opt.part_slots) return false;
    p.dec_deep = !small_tile;
    const int64_t snap = std::max<int64_t>(2, total / W / 16);
    int64_t done = 0, w = 1;                               // cost of the rows so far; workgroup w ends at total * w / W
    p.dec_wg.push_back(0);
    auto next_workgroup = [&] { if ((int32_t)p.dec.size() > p.dec_wg.back()) p.dec_wg.push_back((int32_t)p.dec.size()); };
    for (int s = 0; s < num_seqs; ++s) {
        const SeqMeta& m = p.seqs[s];
        if (m.q_len != 1) continue;
        const int64_t n_pages = (m.ctx_len + kPage - 1) / kPage;
        const size_t first = p.dec.size();
        for (int64_t begin = 0; begin < n_pages;) {
            auto cut = [&] { return total * w / W - done - kItemPages; };     // page of this row at which workgroup w ends
            for (; w < W && cut() <= begin + snap; ++w) next_workgroup();
            if ((int32_t)p.dec.size() - p.dec_wg.back() >= kMaxItemsPerWg) next_workgroup();
            const int64_t end = w < W && cut() < n_pages - snap ? cut() : n_pages;
            p.dec.push_back(DecItem{m.q_off, s, m.ctx_len, (int32_t)begin, (int32_t)end, -1, -1, 0});
            begin = end;
        }
        const int32_t n_split = (int32_t)(p.dec.size() - first);
        if (n_split > 1) {
            p.max_split = std::max(p.max_split, n_split);
            for (int32_t i = 0; i < n_split; ++i) { p.dec[first + i].part = *part + i; p.dec[first + i].cmb = (int32_t)p.cmb.size(); }
            p.cmb.push_back(CmbItem{m.q_off, *part, n_split, 0});
            *part += n_split;
        }
        done += n_pages + kItemPages;
    }
    next_workgroup();
    return true;
}

// Whole rows over the CUs, for launches that are resident at once or nearly so: the memory system serves the CUs alike, so
// what matters is the pages per CU.  Rows go, longest first, to the CU with the least that has room (no CU gets more
// rows than it must); returns the most loaded CU's pages.  order: rows in the order of launch (workgroups are placed
// round-robin: the first rows of all CUs, then the second rows, ...).
// Flat arrays that the plan keeps, and no queue of CUs while they get their first two rows: in the order of the rows'
// lengths the loads are sorted as they are.  (With a queue of (load, CU) pairs and a list per CU, packed once to decide
// and once more for the order, planning a pass took 12.6 us for 88 rows, 16.0 for 128 and 182 for 700 rows of one KV
// head; it takes 2.6, 3.8 and 24.)
static int64_t pack_rows(RowPacking& k, int64_t cus)
{
    const int32_t n = (int32_t)k.pages.size(), n_cu = (int32_t)cus;
    int32_t top = 0;
    for (int32_t x : k.pages) top = std::max(top, x);
    // longest first, equal lengths in batch order (one byte of the length at a time)
    k.by_len.resize(n);
    for (int32_t i = 0; i < n; ++i) k.by_len[i] = i;
    for (int shift = 0; shift < 32 && (top >> shift) > 0; shift += 8) {
        int32_t at[257] = {};
        for (int32_t i : k.by_len) ++at[256 - (k.pages[i] >> shift & 255)];
        for (int v = 1; v <= 256; ++v) at[v] += at[v - 1];
        k.tmp.resize(n);
        for (int32_t i : k.by_len) k.tmp[at[255 - (k.pages[i] >> shift & 255)]++] = i;
        k.by_len.swap(k.tmp);
    }
    const int32_t most = (n + n_cu - 1) / n_cu;            // rows per CU
    k.row.assign((size_t)most * n_cu, -1);                 // [round][CU]
    k.count.assign(n_cu, 0);
    k.load.assign(n_cu, 0);
    int64_t longest = 0;
    auto put = [&](int32_t i, int32_t b) {
        k.row[(size_t)k.count[b]++ * n_cu + b] = i;
        k.load[b] += k.pages[i] + kItemPages;
        longest = std::max(longest, k.load[b]);
    };
    const int32_t n1 = std::min(n, n_cu);
    for (int32_t j = 0; j < n1; ++j) put(k.by_len[j], j);
    if (most == 2) {
        // the CUs by load: from the last one up, equal loads in order of the CUs
        int32_t hi = n_cu, lo = n_cu;
        for (int32_t j = n1, b = n_cu; j < n; ++j, ++b) {
            if (b >= hi) {
                hi = lo;
                for (lo = hi - 1; lo > 0 && k.load[lo - 1] == k.load[hi - 1]; --lo) {}
                b = lo;
            }
            put(k.by_len[j], b);
        }
    } else if (most > 2) {
        // a heap of the CUs with room, least load first (then the CU's number)
        k.open.resize(n_cu);
        for (int32_t b = 0; b < n_cu; ++b) k.open[b] = k.load[b] << 24 | b;
        std::make_heap(k.open.begin(), k.open.end(), std::greater<>());
        int64_t* const h = k.open.data();
        for (int32_t j = n1, left = n_cu; j < n; ++j) {
            const int32_t b = (int32_t)(h[0] & 0xffffff);
            put(k.by_len[j], b);
            const int64_t x = k.count[b] < most ? k.load[b] << 24 | b : h[--left];   // takes the top's place
            int32_t at = 0;
            for (int32_t c = 1; c < left; c = 2 * at + 1) {
                c += c + 1 < left && h[c + 1] < h[c];
                if (h[c] >= x) break;
                h[at] = h[c];
                at = c;
            }
            h[at] = x;
        }
    }
    return longest;
}

// Rows stay whole when the most loaded CU gets at most 24 pages of 8 KB (or as many bytes in smaller ones) more than
// the average: dealing out costs about as much (60 rows of 300-1000 tokens: 36.6 us whole, 41.5 us dealt out; 40 rows
// of 500-1220 tokens, 20 pages over the average: 34.5 against 39.1; 100 rows of 1600-5700 tokens, e4m3, 36 over:
// 155 against 142; 48 rows, head dim 64, 44 over: 62.3 against 57.6).
// They may be as many as decode_kernel_lean has workgroups resident at once (opt.wg_slots; bf16: 1024 with head dim 128,
// 1792 with 64).  The kernel that runs them, decode_kernel_alone, has fewer (768 and 1536): beyond those up to a quarter
// start when the first ones end, and the packing no longer describes where.  The line lies where it does because the
// rules behind it are slower there all the same: whole rows against cut ones, 8 KV heads, bf16: 120 rows of 200-800
// tokens 49.6 us for 56.8, 104 of 400-1600 77.9 for 87.2, 110 of 300-3000 127.2 for 135.0, head dim 64, 216 of 100-900
// 45.9 for 53.3 and 224 of 1000-4000 186.1 for 193.7; 128 of 1000-8000 is the exception, 384.9 for 380.9.
static bool rows_stay_whole(Plan& p, int num_seqs, int64_t pages, const ts_attn_desc& d, const PlanOptions& opt)
{
    const int64_t cus = std::max<int64_t>(1, opt.n_cu / d.num_kv_heads), rows = p.info.decode_tokens;
    if (rows < cus || rows * d.num_kv_heads > opt.wg_slots) return false;
    const int64_t page_bytes = 2 * kPage * d.head_dim * (d.kv_dtype == TS_FP8_E4M3 ? 1 : 2);
    const int64_t most = (pages + rows * kItemPages) / cus + 24 * 8192 / page_bytes;
    p.packing.pages.clear();
    for (int s = 0; s < num_seqs; ++s)
        if (p.seqs[s].q_len == 1) {
            p.packing.pages.push_back((p.seqs[s].ctx_len + kPage - 1) / kPage);
            if (p.packing.pages.back() + kItemPages > most) return false;
        }
    return pack_rows(p.packing, cus) <= most;
}

// The items of rows that stay whole (one per row, in batch order) in the order of launch: CUs with more rows first.
static void order_whole_rows(Plan& p)
{
    const RowPacking& k = p.packing;
    const size_t cus = k.count.size(), most = k.row.size() / cus;
    std::vector<DecItem> packed;
    packed.reserve(p.dec.size());
    for (size_t r = 0; r < most; ++r)
        for (int32_t c = (int32_t)most; c > (int32_t)r; --c)
            for (size_t b = 0; b < cus; ++b)
                if (k.count[b] == c) packed.push_back(p.dec[k.row[r * cus + b]]);
    p.dec.swap(packed);
}

static void sort_decode_items(std::vector<DecItem>& v)
{
    std::stable_sort(v.begin(), v.end(), [](const DecItem& a, const DecItem& b) {
        return (a.page_end - a.page_begin) > (b.page_end - b.page_begin);
    });
}

// Launch order of the prefill workgroups.  Workgroups are dispatched to the accelerator dies
// round-robin (workgroup i runs on die i % xcds) and every die has its own L2.  All tiles of one
// (chunk, KV head) stream read the same K/V pages, so a stream is pinned to one die and its tiles
// are launched next to each other: they walk the stream's pages almost in step, and the pages are
// fetched from HBM about once instead of once per tile.  Streams are spread over the dies by
// decreasing work (greedy), longest tiles of a stream first.
// A die with at most two tiles per CU whose streams' K/V stay in its 4 MB of L2 anyway (kDieResidentBytes) launches
// its tiles longest first instead: by streams, the later streams' long tiles come last and set the time.  8 prompts
// of 128-512 tokens (1.5 tiles per CU) 33.9 -> 30.6 us, 16 of 64-256 (1.25) 32.4 -> 29.3; with more tiles the dispatch
// evens out by itself and the order by streams is the better one: 8 prompts of 512-1024 tokens (3 tiles per CU)
// 81 us, longest first 84; 16 of them 143 against 153.
constexpr int64_t kDieResidentBytes = 2 << 20;
constexpr size_t kLongestFirstTilesPerCu = 2;
static int64_t pf_keys(const PfItem& t)
{
    return std::min(t.prefix + t.tok_begin + t.tok_count, t.kv_end) - t.kv_begin;
}

// Parts of a tile that is cut along the keys (`below`: keys at or below its first query position that may be cut off): one per
// shortest range ...
static int32_t parts_in_ranges(int32_t below, int32_t min_keys, int32_t wanted)
{
    return min_keys > 0 ? std::max(1, std::min(wanted, below / min_keys)) : 1;
}
// ... or, where half_ranges_pay, four parts of half the shortest range before five or more of it, and nothing below one and a half.
// Up to four are merged by the last of them, about 5 us on top of a tile whose 64 keys take 1-1.5 us; more by a launch, as
// much again.  One part per range and four halves: 32 tokens over 1000 29.1 and 24.8 us a pass, 128 over 1500 31.2 and
// 27.0, 400 over 1000 (head dim 64) 24.5 and 21.0, 128 over 2700 (five parts) 36.2 and 31.1; from six ranges on the launch:
// 32 over 4200 32.7 against 35.6 in four parts.  Whole below 768 keys: 32 over 500 in two parts 22.7 against 20.6.
constexpr int32_t kPfLaunchParts = 6;
static int32_t parts_of_tile(int32_t below, int32_t min_keys, int32_t wanted)
{
    if (below / min_keys >= kPfLaunchParts) return std::min(wanted, below / min_keys);
    if (2 * (int64_t)below < 3 * (int64_t)min_keys) return 1;
    return std::max(1, std::min({wanted, kPfMergeParts, (int32_t)(2 * (int64_t)below / min_keys)}));
}
// Halves do not pay
//   - where some tile goes into more than four parts: a merge is launched anyway (32/8 heads, e4m3, 3 chunks of 7-30 over 2645-5403
//     42.0 us with halves, 34.2 in ranges);
//   - where a die has not a CU for each: in a launch of its own the tiles of a (sequence, head) stream stay on one die, so
//     with few KV heads some dies fill while others are idle (64/4 heads, chunks of 106 and 339 over 993, 44 pieces on a die, 46.6
//     and 33.7; 16/2, 900 over 800, 95 pieces, 65.5 and 52.1; 28/4, 3 chunks of 172-300 over 828-2418 39.4 and 34.1; but 8/4,
//     1164-1645 alone, 30 pieces, 27.8 and 32.9) -- unless ranges would come to a launch (4/2, 1306-2152 over 715-1446, 48.5 and 57.1);
//   - in two parts over a bf16 cache, where nearly every CU has a tile as it is (3 chunks of 294-327 over 885-1026 34.0 and 32.0,
//     430-856 over 705-823 33.3 and 32.2; e4m3 gains: 3 of 767-1187, 8/8 heads, 31.3 and 35.4).
// (parts_of_tile grows with the keys: a sequence's last tile has the most parts)
static bool half_ranges_pay(const Plan& p, int num_seqs, int32_t TT, int Hkv, int32_t kv_dtype, const PlanOptions& opt, int32_t min_keys,
                            int32_t wanted, bool pinned)
{
    if (wanted < 3 && kv_dtype != TS_FP8_E4M3) return false;
    const int64_t xcds = std::max(1, opt.xcds);
    int64_t chunks = 0, pieces = 0;                        // pieces of the stream that has most
    int32_t most = 1, ranges = 1;
    for (int s = 0; s < num_seqs; ++s) {
        const SeqMeta& m = p.seqs[s];
        if (m.q_len <= 1) continue;
        const int32_t last = (m.prefix + (m.q_len - 1) / TT * TT) / 64 * 64;
        chunks += 1;
        most = std::max(most, parts_of_tile(last, min_keys, wanted));
        ranges = std::max(ranges, parts_in_ranges(last, min_keys, wanted));
        if (!pinned || Hkv % xcds == 0) continue;          // (as many KV heads as dies: `wanted` parts a tile have a CU each)
        int64_t n = 0;
        for (int32_t t0 = 0; t0 < m.q_len; t0 += TT) n += parts_of_tile((m.prefix + t0) / 64 * 64, min_keys, wanted);
        pieces = std::max(pieces, n);
    }
    if (most > kPfMergeParts) return false;
    return ranges > kPfMergeParts || (chunks * Hkv + xcds - 1) / xcds * pieces <= opt.n_cu / xcds;
}

// Do the tiles over an e4m3 cache gain by bf16 copies of their pages, or do they convert while they stage?  The copies cost a
// launch and three bytes of traffic per element in front of everything else, decode rows included; converting costs a tile
// 4-8 % of every stage.  So it depends on how often a page is read.  Whole passes, converting against copies, 8 KV heads:
// 4 chunks of 64 over 8200 (1-2 reads a page) 51.5 us against 82.3; 8 of 256 over 8200 (4) 250 against 301; 512 over 8200 (16)
// 136.1 against 140.3; 512 over 8200 next to 128 rows of 1-8 Ki tokens 310 against 335; 1024 over 4000 (29) next to 400 rows
// 267 against 262; 4 of 1024 over 8200 (30) 996 against 974; 2048 over 8200 (57) 530 against 511.  Few pages: the copies are a
// few microseconds and the tile's first stages arrive later where they are converted: one chunk of 512 alone (32 pages) 23.4
// against 22.8, of 32 16.0 against 13.2; 32 over 1000 (65 pages) 31.7 against 31.6; 8 of 256 (128 pages) 33.8 against 36.2.
constexpr int64_t kWidenReads = 26;
constexpr int64_t kWidenFewPages = 512;                    // (pages times KV heads)
// Where one tile's chain of stages sets the time (it is kWidenChain times a CU's share of all stages: long prompts, few heads),
// converting is paid on every one of them while most CUs have nothing to hide it behind, and the copies only once.  One prompt of
// 6000 tokens with 8/8 heads (12 reads a page, 94 stages) 138.3 us converting, 129.8 with copies, of 7800 with 8/4 heads 138.7 and 131.4;
// two of 8700 with 4/4 heads 204.7 and 194.1; of 3000 tokens with 8/8 heads (cut in two) 49.2 and 51.8.  Over 120 prefill batches below the
// line of reads: converting always 0.6 % over the better one on average (6 % at most), so 0.2 % (2 % but for five of 29-100 us).
constexpr double kWidenChain = 1.4, kWidenStageUs = 0.2, kWidenLaunchUs = 4.0, kWidenPageUs = 12288 / 4.5e6;   // (4 KB read, 8 written)
static bool widening_pays(const Plan& p, int64_t pages, int Hkv, int32_t n_cu)
{
    if (pages * Hkv < kWidenFewPages) return true;
    int64_t keys = 0, longest = 0;                         // that tiles read, per KV head; by the longest tile or part
    for (const PfItem& t : p.pf) { keys += pf_keys(t); longest = std::max(longest, pf_keys(t)); }
    if (p.info.decode_tokens == 0 && longest * n_cu > kWidenChain * keys * Hkv &&
        kWidenStageUs * longest / 64 > kWidenLaunchUs + (double)pages * Hkv * kWidenPageUs) return true;
    return keys > kWidenReads * kPage * pages;
}

static void map_prefill_to_xcds(Plan& p, int Hkv, int xcds, int mixed_mode, bool for_launch, int64_t kv_row_bytes,
                                int32_t n_cu)
{
    if (p.pf.empty()) return;
    const bool queued = mixed_mode != TS_MIXED_SEPARATE && !p.dec.empty();
    // the tiles sequence by sequence, longest first (p.pf is sorted longest first, the stable sort keeps that)
    std::vector<int32_t> tiles(p.pf.size());
    for (size_t i = 0; i < tiles.size(); ++i) tiles[i] = (int32_t)i;
    std::stable_sort(tiles.begin(), tiles.end(), [&](int32_t a, int32_t b) { return p.pf[a].seq < p.pf[b].seq; });
    struct Stream { int32_t begin, end, g; int64_t work; };        // tiles[begin, end) of one sequence, for one KV head
    std::vector<Stream> streams;
    for (size_t i = 0, j; i < tiles.size(); i = j) {
        int64_t work = 0;
        for (j = i; j < tiles.size() && p.pf[tiles[j]].seq == p.pf[tiles[i]].seq; ++j) work += pf_keys(p.pf[tiles[j]]);
        for (int g = 0; g < Hkv; ++g) streams.push_back(Stream{(int32_t)i, (int32_t)j, g, work});
    }
    std::stable_sort(streams.begin(), streams.end(), [](const Stream& a, const Stream& b) { return a.work > b.work; });
    std::vector<std::vector<Stream>> on(xcds);
    std::vector<int64_t> load(xcds, 0);
    std::vector<size_t> n_tiles(xcds, 0);
    for (const Stream& st : streams) {
        const size_t best = std::min_element(load.begin(), load.end()) - load.begin();
        load[best] += st.work;
        n_tiles[best] += st.end - st.begin;
        on[best].push_back(st);
    }
    // the die's (tile, head) pairs in launch order
    auto tiles_of = [&](int x) {
        std::vector<PfSlot> v;
        int64_t keys = 0;
        for (const Stream& st : on[x]) {
            keys += p.pf[tiles[st.begin]].ctx_len;
            for (int32_t t = st.begin; t < st.end; ++t) v.push_back(PfSlot{tiles[t], st.g});
        }
        if (v.size() <= kLongestFirstTilesPerCu * (size_t)(n_cu / xcds) && keys * kv_row_bytes <= kDieResidentBytes)
            std::stable_sort(v.begin(), v.end(), [&](const PfSlot& a, const PfSlot& b) { return pf_keys(p.pf[a.item]) > pf_keys(p.pf[b.item]); });
        return v;
    };
    if (!(for_launch && queued)) {
        p.pfmap.assign(*std::max_element(n_tiles.begin(), n_tiles.end()) * xcds, PfSlot{-1, 0});
        for (int x = 0; x < xcds; ++x) {
            size_t k = x;
            for (const PfSlot& t : tiles_of(x)) { p.pfmap[k] = t; k += xcds; }
        }
    }
    if (!queued) return;
    if (mixed_mode == TS_MIXED_CORESIDENT) {
        // The tiles alone, die by die in the launch order above, for the resident prefill workgroups; the
        // decode items run as a grid of their own next to them.
        p.q_off.assign(xcds + 1, 0);
        for (int x = 0; x < xcds; ++x) {
            for (const PfSlot& t : tiles_of(x)) p.queue.push_back(QItem{t.item << 1 | 1, t.head_kv});
            p.q_off[x + 1] = (int32_t)p.queue.size();
        }
        return;
    }
    std::vector<std::vector<PfSlot>> per(xcds);
    for (int x = 0; x < xcds; ++x)
        for (const Stream& st : on[x])
            for (int32_t t = st.begin; t < st.end; ++t) per[x].push_back(PfSlot{tiles[t], st.g});

    // Mixed batch: one queue per die for the persistent kernel.  Decode items (HBM-bound) and
    // prefill tiles (MFMA-bound) are interleaved by their share of their own kind's total cost, so
    // that both kinds are in flight on every CU from the first to the last item and finish together.
    std::vector<std::vector<PfSlot>> dper(xcds);
    {
        int64_t j = 0;
        for (size_t i = 0; i < p.dec.size(); ++i)
            for (int g = 0; g < Hkv; ++g, ++j) dper[j % xcds].push_back(PfSlot{(int32_t)i, g});
    }
    p.q_off.assign(xcds + 1, 0);
    for (int x = 0; x < xcds; ++x) {
        double dtot = 0, ptot = 0;
        for (const PfSlot& d : dper[x]) dtot += p.dec[d.item].page_end - p.dec[d.item].page_begin;
        for (const PfSlot& t : per[x]) ptot += pf_keys(p.pf[t.item]);
        size_t di = 0, ti = 0;
        double dacc = 0, pacc = 0;
        while (di < dper[x].size() || ti < per[x].size()) {
            const double dkey = di < dper[x].size() ? dacc / std::max(1.0, dtot) : 2.0;
            const double pkey = ti < per[x].size() ? pacc / std::max(1.0, ptot) : 2.0;
            if (dkey <= pkey) {                            // decode first on ties (Sec. 4.5.2)
                const PfSlot& d = dper[x][di++];
                dacc += p.dec[d.item].page_end - p.dec[d.item].page_begin;
                p.queue.push_back(QItem{d.item << 1, d.head_kv});
            } else {
                const PfSlot& t = per[x][ti++];
                pacc += pf_keys(p.pf[t.item]);
                p.queue.push_back(QItem{t.item << 1 | 1, t.head_kv});
            }
        }
        p.q_off[x + 1] = (int32_t)p.queue.size();
    }
}

void Plan::clear()
{
    seqs.clear(); dec.clear(); dec_wg.clear(); cmb.clear(); pf.clear(); pfcmb.clear(); pfmap.clear(); apt.clear(); apr.clear();
    queue.clear(); q_off.clear(); rt.clear(); rtcut.clear(); wide.clear(); wide_base.clear();
    dec_deep = pf_merge_launch = false;
    max_split = 1;
    info = ts_plan_info{};
}

void build_plan(const ts_attn_desc& d, const int32_t* q_lens, const int32_t* ctx_lens, int num_seqs,
                const PlanOptions& options, Plan* plan)
{
    PlanOptions opt = options;
    if (opt.wg_slots <= 0) opt.wg_slots = decode_places_per_cu(d.head_dim) * std::max(1, opt.n_cu);
    Plan& p = *plan;
    p.clear();
    const bool mfma = desc_uses_mfma(d) && !opt.generic_only;
    const bool mfma_dec = desc_uses_mfma_decode(d) && !opt.generic_only;
    // fp8 caches: can the pages of the chunks' sequences be widened to bf16 for this pass (see below)?
    int64_t chunk_pages = 0;
    for (int s = 0; s < num_seqs; ++s)
        if (q_lens[s] > 1) chunk_pages += (ctx_lens[s] + kPage - 1) / kPage;
    const bool widen = d.kv_dtype == TS_FP8_E4M3 && chunk_pages > 0 && opt.widen_pages > 0 && chunk_pages <= opt.widen_pages;
    // Chunk rows run as matrix-core tiles; with head dim 64 the tiles read bf16 pages only (a bf16 cache, or the
    // widened copies of an e4m3 cache), otherwise the rows go to the generic kernel.
    const bool mfma_tiles = desc_uses_mfma_tiles(d) && !opt.generic_only && !opt.prefill_generic &&
                            (d.head_dim == 128 || d.kv_dtype == TS_BF16 || widen);
    const int Hkv = d.num_kv_heads;
    int64_t rt_tokens = 0;                                 // rows the generic kernel gets
    p.seqs.resize((size_t)num_seqs + 1);
    int32_t off = 0;
    int64_t decode_tiles = 0, decode_pages = 0;
    for (int s = 0; s < num_seqs; ++s) {
        p.seqs[s] = SeqMeta{off, q_lens[s], ctx_lens[s], ctx_lens[s] - q_lens[s]};
        off += q_lens[s];
        p.info.ctx_pages += (ctx_lens[s] + kPage - 1) / kPage;
        if (q_lens[s] == 1) {
            p.info.decode_tokens += 1;
            decode_pages += (ctx_lens[s] + kPage - 1) / kPage;
            decode_tiles += (int64_t)((ctx_lens[s] + kPage - 1) / kPage) * Hkv;
        } else {
            p.info.prefill_tokens += q_lens[s];
        }
    }
    p.seqs[num_seqs] = SeqMeta{off, 0, 0, 0};
    p.info.total_tokens = off;

    // append work: chunks page by page where the page-wise kernel applies, the rest token by token
    const bool page_wise = d.q_dtype == TS_BF16 && d.kv_dtype != TS_F32 && (d.head_dim == 128 || d.head_dim == 64);
    for (int s = 0; opt.append_lists && s < num_seqs; ++s) {
        const SeqMeta& m = p.seqs[s];
        if (!page_wise || m.q_len < kAppendTileMin) {
            for (int32_t i = 0; i < m.q_len; ++i) {
                const int32_t pos = m.prefix + i;
                const bool leads = d.kv_dtype == TS_F32 && (i == 0 || pos % kPage == 0);
                if (opt.for_launch && d.kv_dtype == TS_F32 && !leads) continue;   // (the run's first record stands for it)
                p.apr.push_back(AppRow{m.q_off + i, s, pos, leads ? std::min(kPage - pos % kPage, m.q_len - i) : 0});
            }
            continue;
        }
        for (int32_t pg = m.prefix / kPage; pg <= (m.ctx_len - 1) / kPage; ++pg) {
            const int32_t lo = std::max(m.prefix, pg * kPage) - pg * kPage;
            const int32_t hi = std::min(m.ctx_len, (pg + 1) * kPage) - pg * kPage;
            p.apt.push_back(AppTile{s, pg, lo | hi << 8, m.q_off + pg * kPage - m.prefix});
        }
    }

    if (opt.append_only) return;
    const int32_t TT = opt.tile_tokens > 0 ? opt.tile_tokens : prefill_tile_tokens(d);
    int64_t tile_heads = 0;                                // prefill workgroups of the batch
    if (mfma_tiles)
        for (int s = 0; s < num_seqs; ++s)
            if (p.seqs[s].q_len > 1) tile_heads += (int64_t)((p.seqs[s].q_len + TT - 1) / TT) * Hkv;
    // How a batch with both kinds of rows is launched.  Co-resident by default; class by class when either class
    // is too short for the overlap to pay for the fork and join (kCoresidentMinUs).
    int mixed_mode = opt.mixed_mode;
    int32_t longest = 0;                                   // keys of the longest tile
    for (int s = 0; s < num_seqs; ++s)
        if (p.seqs[s].q_len > 1) longest = std::max(longest, p.seqs[s].ctx_len);
    double t_pf = 0, t_dec = 0;                            // microseconds each kind would take alone
    if (mixed_mode == TS_MIXED_CORESIDENT) {
        double flop = 0;
        for (int s = 0; s < num_seqs; ++s) {
            const SeqMeta& m = p.seqs[s];
            if (m.q_len > 1) flop += 4.0 * d.num_q_heads * d.head_dim * ((double)m.q_len * m.prefix + 0.5 * m.q_len * (m.q_len + 1.0));
        }
        t_pf = flop / kPfFlopPerUs;
        t_dec = (double)decode_tiles * 2.0 * kPage * d.head_dim * (d.kv_dtype == TS_FP8_E4M3 ? 1 : 2) / kDecBytePerUs;
        // (a stated number of resident workgroups asks for this launch form whatever the batch)
        if (opt.pf_resident_wgs <= 0 && std::min(t_pf, t_dec) < kCoresidentMinUs) mixed_mode = TS_MIXED_SEPARATE;
    }
    if (!mfma || p.info.decode_tokens == 0 || tile_heads == 0) mixed_mode = TS_MIXED_SEPARATE;
    if (!mfma_dec) { decode_tiles = 0; decode_pages = 0; }
    p.info.mixed_mode = mixed_mode;
    // Co-resident launch: how many CUs get a resident prefill workgroup.  Such a CU has room for one decode
    // workgroup instead of four, so a batch whose decode scan outlasts its tiles (one restricted chunk next to a
    // large decode batch, Sec. 4.4) keeps part of the CUs for decode rows alone: the tiles get a share of the CUs
    // that grows with the ratio of the two times (estimated from the batch's flops and bytes at the rates the
    // kernels reach alone), in multiples of the number of dies.
    int32_t pf_wgs = 0;
    if (mixed_mode == TS_MIXED_CORESIDENT) {
        const int32_t x = std::max(1, opt.xcds);
        const int32_t all = std::max(1, opt.n_cu);
        if (opt.pf_resident_wgs > 0) {
            pf_wgs = std::min(all, opt.pf_resident_wgs);
        } else {
            const double r = t_dec > 0 ? t_pf / t_dec : 1e9;
            const bool wide = d.num_q_heads > 8 * d.num_kv_heads, bf16 = d.kv_dtype == TS_BF16, short_scan = t_dec < kPfAllUs;
            const bool every = r >= (short_scan ? (bf16 ? kPfAllRatioShort : kPfAllRatioShort8) : wide ? kPfAllRatioWide : kPfAllRatio);
            double share = kPfShare0 + kPfShare1 * r;
            if (bf16 && short_scan) share = std::max(share, kPfShort0 + kPfShort1 * r);
            else if (bf16) share = wide ? kPfShare0Wide + kPfShare1Wide * r : std::max(share, kPfSteep0 + kPfSteep1 * r);
            pf_wgs = every ? all : (int32_t)std::ceil(share * all);
            // (not a few tiles more than whole rounds: 55 tiles per die on 19 workgroups 485 us, on 18 509)
            const int64_t per_die = (tile_heads + x - 1) / x, n = (pf_wgs + x - 1) / x, rounds = per_die / n;
            if (rounds > 0 && per_die % n > 0 && per_die % n <= n / 8) pf_wgs = (int32_t)((per_die + rounds - 1) / rounds * x);
        }
        pf_wgs = std::min(all, std::max(x, (pf_wgs + x - 1) / x * x));
    }
    const bool filled_by_prefill = mixed_mode != TS_MIXED_SEPARATE && (tile_heads >= opt.n_cu || pf_wgs > 0);
    const int32_t L = opt.split_pages > 0
                          ? opt.split_pages
                          : auto_split_pages(p, num_seqs, decode_tiles, decode_pages, Hkv, opt.wg_slots,
                                             std::max(1, opt.n_cu), filled_by_prefill, pf_wgs, t_pf,
                                             d.num_q_heads > 8 * d.num_kv_heads && d.kv_dtype == TS_BF16);
    // (rows up to this many pages stay whole: see 4. above)
    const bool many = mixed_mode == TS_MIXED_SEPARATE && p.info.decode_tokens * Hkv > opt.wg_slots;
    const int32_t keep_whole = opt.split_pages > 0 || !many ? L : L + L / 4;
    p.info.split_pages = keep_whole;
    p.info.tile_tokens = TT;

    int32_t part = 0, pf_part = 0;
    // rows that give every CU a workgroup and come out even over the CUs stay whole; else they are dealt out evenly
    const bool whole = mfma_dec && opt.split_pages == 0 && mixed_mode == TS_MIXED_SEPARATE && rows_stay_whole(p, num_seqs, decode_pages, d, opt);
    const bool even = mfma_dec && !whole && opt.split_pages == 0 && mixed_mode == TS_MIXED_SEPARATE &&
                      deal_decode_evenly(p, num_seqs, decode_pages, d, opt, &part);
    // parts per prefill tile that would give every CU a workgroup (1 = the tiles fill the GPU as they are)
    // (next to a scan that outlasts the longest tile there is nothing to gain: 512 tokens over 4096 next to 128 rows 416 us
    // whole, 428 in two parts)
    const bool parts_pay = mixed_mode != TS_MIXED_CORESIDENT || kStageUs * longest / 64 > t_dec;
    const int64_t pf_parts_wanted = tile_heads > 0 && parts_pay ? std::min<int64_t>(16, (pf_wgs > 0 ? pf_wgs : opt.n_cu) / tile_heads) : 1;
    const int32_t min_keys = pf_parts_wanted > 1 ? opt.pf_split_min_keys : 0, most_parts = (int32_t)pf_parts_wanted;
    const bool halves = min_keys > 0 && half_ranges_pay(p, num_seqs, TT, Hkv, d.kv_dtype, opt, min_keys, most_parts, mixed_mode == TS_MIXED_SEPARATE);
    for (int s = 0; s < num_seqs; ++s) {
        const SeqMeta& m = p.seqs[s];
        if (m.q_len == 0) continue;
        const bool as_decode = mfma_dec && m.q_len == 1;
        const bool as_tiles = mfma_tiles && m.q_len > 1;
        if (as_decode && even) continue;
        if (as_decode) {
            int32_t n_pages = (m.ctx_len + kPage - 1) / kPage;
            int32_t n_split = whole || n_pages <= keep_whole ? 1 : (n_pages + L - 1) / L;
            int32_t per = (n_pages + n_split - 1) / n_split;
            n_split = (n_pages + per - 1) / per;
            const int32_t cmb_idx = n_split > 1 ? (int32_t)p.cmb.size() : -1;
            p.max_split = std::max(p.max_split, n_split);
            if (n_split > 1) p.cmb.push_back(CmbItem{m.q_off, part, n_split, 0});
            for (int32_t k = 0; k < n_split; ++k) {
                int32_t b = k * per, e = std::min(n_pages, b + per);
                p.dec.push_back(DecItem{m.q_off, s, m.ctx_len, b, e, n_split > 1 ? part + k : -1, cmb_idx, 0});
            }
            if (n_split > 1) part += n_split;
        } else if (as_tiles) {
            for (int32_t t0 = 0; t0 < m.q_len; t0 += TT) {
                const int32_t cnt = std::min(TT, m.q_len - t0);
                // Cut along the keys when the batch's tiles cannot occupy the GPU (a short chunk over a long
                // prefix -- the one-task-at-a-time shape of Sec. 4.4 -- walks thousands of keys in a handful of
                // workgroups otherwise).  Cuts lie at multiples of 64 keys at or below the tile's first query
                // position, so that every row sees the first key of every part; parts are of equal length.
                const int32_t below = (m.prefix + t0) / 64;                       // whole stages every row sees fully
                const int32_t n_part = halves ? parts_of_tile(below * 64, min_keys, most_parts) : parts_in_ranges(below * 64, min_keys, most_parts);
                if (n_part == 1) {
                    p.pf.push_back(PfItem{s, m.q_off, m.q_len, m.prefix, t0, cnt, m.ctx_len, -1, 0, INT32_MAX, 0, 0});
                    continue;
                }
                const int32_t total = (m.prefix + t0 + cnt + 63) / 64;            // stages of the whole tile
                const int32_t per = (total + n_part - 1) / n_part;
                int32_t begin = 0, made = 0;
                const int32_t first = pf_part;
                for (int32_t cut = per; cut <= below && cut < total; cut += per, ++made) {
                    p.pf.push_back(PfItem{s, m.q_off, m.q_len, m.prefix, t0, cnt, m.ctx_len, pf_part++, begin * 64, cut * 64, 0, 0});
                    begin = cut;
                }
                if (made == 0) {                                                   // no admissible cut after all
                    p.pf.push_back(PfItem{s, m.q_off, m.q_len, m.prefix, t0, cnt, m.ctx_len, -1, 0, INT32_MAX, 0, 0});
                    continue;
                }
                p.pf.push_back(PfItem{s, m.q_off, m.q_len, m.prefix, t0, cnt, m.ctx_len, pf_part++, begin * 64, INT32_MAX, 0, 0});
                ++made;
                p.pfcmb.push_back(PfCmb{(int32_t)p.pf.size() - made, first, made, 0});
                // (the lists are exported without this launch detail; the counters hold n_cu words: cut tiles are
                // fewer than half the CUs)
                if (opt.for_launch && made <= kPfMergeParts && (int64_t)p.pfcmb.size() * Hkv <= opt.n_cu) {
                    p.pfcmb.back().in_kernel = 1;
                    for (int32_t k = 1; k <= made; ++k) p.pf[p.pf.size() - k].merge = (int32_t)p.pfcmb.size();
                } else {
                    p.pf_merge_launch = true;
                }
            }
        } else {
            const int32_t TR = row_tile_tokens(d);
            for (int32_t i = 0; i < m.q_len; i += TR) {
                const int32_t cnt = std::min(TR, m.q_len - i);
                p.rt.push_back(RowTile{s, m.q_off + i, m.prefix + i, cnt});
            }
            rt_tokens += m.q_len;
        }
    }
    if (!p.rt.empty()) part = cut_row_tiles(p, d.num_q_heads / Hkv, Hkv, opt, part);
    // fp8 caches: the pages of the chunks' sequences are widened to bf16 once per pass, provided they fit the scratch the
    // option allows and the pass gains by it (see widening_pays)
    if (widen && !p.pf.empty() && (d.head_dim != 128 || widening_pays(p, chunk_pages, Hkv, opt.n_cu))) {
        p.wide_base.assign((size_t)num_seqs, -1);
        for (int s = 0; s < num_seqs; ++s) {
            if (p.seqs[s].q_len <= 1) continue;
            p.wide_base[s] = (int32_t)p.wide.size();
            const int32_t n_pages = (p.seqs[s].ctx_len + kPage - 1) / kPage;
            for (int32_t j = 0; j < n_pages; ++j) p.wide.push_back(WideItem{s, j});
        }
    }
    p.info.widened_pages = (int64_t)p.wide.size();
    // longest first (stable, so equal lengths keep batch order and runs stay reproducible)
    if (whole) order_whole_rows(p);
    else if (!even) sort_decode_items(p.dec);
    {
        // (the merge list refers to the tiles by position: sort a permutation and carry the references along)
        std::vector<int32_t> order(p.pf.size()), where(p.pf.size());
        for (size_t i = 0; i < order.size(); ++i) order[i] = (int32_t)i;
        std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return pf_keys(p.pf[a]) > pf_keys(p.pf[b]); });
        std::vector<PfItem> sorted(p.pf.size());
        for (size_t i = 0; i < order.size(); ++i) { sorted[i] = p.pf[order[i]]; where[order[i]] = (int32_t)i; }
        p.pf.swap(sorted);
        for (PfCmb& cm : p.pfcmb) cm.item = where[cm.item];
    }
    map_prefill_to_xcds(p, Hkv, std::max(1, opt.xcds), mixed_mode, opt.for_launch, 2 * 2 * d.head_dim, opt.n_cu);
    std::stable_sort(p.rt.begin(), p.rt.end(), [&](const RowTile& a, const RowTile& b) {
        return row_tile_pages(p, a) > row_tile_pages(p, b);
    });
    p.info.n_decode_items = (int32_t)p.dec.size();
    for (const DecItem& it : p.dec) p.info.split_pages = std::max(p.info.split_pages, it.page_end - it.page_begin);
    p.info.n_combine_rows = (int32_t)p.cmb.size();
    p.info.n_prefill_tiles = (int32_t)p.pf.size();
    p.info.n_generic_rows = (int32_t)rt_tokens;
    p.info.partial_slots = part;
    p.info.prefill_parts = pf_part;
    p.info.prefill_workgroups = (int32_t)std::min<int64_t>(pf_wgs, (int64_t)p.queue.size());
}

}  // namespace ts

// ---- host-only C entry points -------------------------------------------------------------------

extern "C" int ts_check_desc(const ts_attn_desc* desc)
{
    return ts::check_desc_impl(desc, nullptr);
}

namespace ts { int check_desc_msg(const ts_attn_desc* d, std::string* err) { return check_desc_impl(d, err); } }

extern "C" int64_t ts_cache_bytes(const ts_attn_desc* d)
{
    if (ts::check_desc_impl(d, nullptr) != TS_OK) return 0;
    int64_t es = d->kv_dtype == TS_F32 ? 4 : (d->kv_dtype == TS_BF16 ? 2 : 1);
    return d->num_pages * d->num_kv_heads * ts::kPage * d->head_dim * es;
}

extern "C" int ts_plan_describe(const ts_attn_desc* desc, const int32_t* q_lens, const int32_t* ctx_lens,
                                int num_seqs, int32_t split_pages, ts_plan_info* out)
{
    std::string err;
    int rc = ts::check_desc_impl(desc, &err);
    if (rc != TS_OK) return rc;
    if (!out || split_pages < 0) return TS_ERR_INVALID_ARG;
    rc = ts::validate_batch(*desc, q_lens, ctx_lens, num_seqs, &err);
    if (rc != TS_OK) return rc;
    ts::Plan plan;
    ts::PlanOptions opt;
    opt.split_pages = split_pages;
    ts::build_plan(*desc, q_lens, ctx_lens, num_seqs, opt, &plan);
    *out = plan.info;
    return TS_OK;
}

extern "C" int64_t ts_plan_export(const ts_attn_desc* desc, const int32_t* q_lens, const int32_t* ctx_lens,
                                  int num_seqs, int32_t split_pages, int32_t wg_slots, int32_t mixed_mode, int which,
                                  int32_t* out, int64_t capacity)
{
    std::string err;
    int rc = ts::check_desc_impl(desc, &err);
    if (rc != TS_OK) return rc;
    if (split_pages < 0 || wg_slots < 0 || capacity < 0 || (capacity > 0 && !out)) return TS_ERR_INVALID_ARG;
    if (mixed_mode < -1 || mixed_mode > TS_MIXED_CORESIDENT) return TS_ERR_INVALID_ARG;
    rc = ts::validate_batch(*desc, q_lens, ctx_lens, num_seqs, &err);
    if (rc != TS_OK) return rc;
    ts::Plan plan;
    ts::PlanOptions opt;
    opt.split_pages = split_pages;
    if (wg_slots > 0) opt.wg_slots = wg_slots;
    if (mixed_mode >= 0) opt.mixed_mode = mixed_mode;
    ts::build_plan(*desc, q_lens, ctx_lens, num_seqs, opt, &plan);
    const void* src = nullptr;
    int64_t n = 0, words = 0;
    std::vector<std::array<int32_t, 4>> rows;              // lists whose records are packed on the device
    if (which == TS_LIST_ROWS) {
        for (const ts::RowTile& t : plan.rt)
            for (int32_t i = 0; i < (t.n_tok_cut & 255) && (t.n_tok_cut < 256 || plan.rtcut[(t.n_tok_cut >> 8) - 1].page_begin == 0); ++i) rows.push_back({t.row0 + i, t.seq, t.pos0 + i + 1, 0});
        std::stable_sort(rows.begin(), rows.end(), [](const std::array<int32_t, 4>& a, const std::array<int32_t, 4>& b) {
            return a[2] != b[2] ? a[2] > b[2] : a[0] < b[0];
        });
    }
    switch (which) {
    case TS_LIST_DECODE:
        ts::sort_decode_items(plan.dec);                    // (dealt out evenly they are listed workgroup by workgroup)
        src = plan.dec.data();   n = (int64_t)plan.dec.size();   words = sizeof(ts::DecItem) / 4; break;
    case TS_LIST_COMBINE: src = plan.cmb.data();   n = (int64_t)plan.cmb.size();   words = sizeof(ts::CmbItem) / 4; break;
    case TS_LIST_PREFILL: src = plan.pf.data();    n = (int64_t)plan.pf.size();    words = sizeof(ts::PfItem) / 4; break;
    case TS_LIST_PFMAP:   src = plan.pfmap.data(); n = (int64_t)plan.pfmap.size(); words = sizeof(ts::PfSlot) / 4; break;
    case TS_LIST_ROWS:    src = rows.data();       n = (int64_t)rows.size();       words = 4; break;
    case TS_LIST_QUEUE:
        for (const ts::QItem& q : plan.queue) rows.push_back({q.item_kind & 1, q.item_kind >> 1, q.head_kv, 0});
        src = rows.data();       n = (int64_t)rows.size();       words = 4; break;
    case TS_LIST_QOFF:    src = plan.q_off.data(); n = (int64_t)plan.q_off.size(); words = 1; break;
    case TS_LIST_APPEND:
        for (const ts::AppTile& t : plan.apt) {
            rows.push_back({t.seq, t.page_idx, t.slots & 255, t.slots >> 8});
            rows.push_back({t.row_slot0, 0, 0, 0});
        }
        src = rows.data();       n = (int64_t)rows.size() / 2;   words = 8; break;
    case TS_LIST_APPEND_ROWS:
        for (ts::AppRow& r : plan.apr) r.run = 0;           // (launch detail)
        src = plan.apr.data(); n = (int64_t)plan.apr.size(); words = sizeof(ts::AppRow) / 4; break;
    case TS_LIST_PFCOMBINE: src = plan.pfcmb.data(); n = (int64_t)plan.pfcmb.size(); words = sizeof(ts::PfCmb) / 4; break;
    case TS_LIST_WIDEN:   src = plan.wide.data();  n = (int64_t)plan.wide.size();  words = sizeof(ts::WideItem) / 4; break;
    default: return TS_ERR_INVALID_ARG;
    }
    const int64_t fit = words ? std::min<int64_t>(n, capacity / words) : 0;
    if (fit > 0) memcpy(out, src, (size_t)(fit * words) * 4);
    return n;
}
