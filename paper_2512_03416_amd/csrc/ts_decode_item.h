// Step a2: decode attention over the paged cache, as a device function shared by the decode
// kernel and the persistent mixed kernel.
//
// A decode row reads its whole cached context once and does ~2*G flops per cache element, so
// the scan is bound by HBM bandwidth (the paper's "memory-intensive decode" whose spare compute
// lets a decoder absorb prefill work, Sec. 1, Sec. 3.4).  The kernel is therefore built around
// the loads:
//   - one workgroup of 4 wavefronts owns one item = (decode row, KV head, page range), the waves
//     taking every 4th page; they share nothing until the end of the item, so many independent
//     waves per CU keep loads in flight;
//   - every (page, KV head) tile is one contiguous 4 KB (bf16) / 2 KB (fp8) block; each load
//     instruction of the wave reads a contiguous 1 KB (K) or 512 B / 256 B (V) run of it, already
//     in matrix-operand order, straight into registers;
//   - NBUF tiles are in flight per wave (register ring, unconditional prefetch so the hardware
//     load counter is statically known);
//   - the G query heads of the KV head's group ride along as columns of the same MFMA
//     (S^T = K Q^T, 16 tokens x 16 columns), so each K/V byte is loaded once for the group;
//   - the accumulator layout of S^T is the B-operand layout of the next MFMA (O^T += V^T P^T),
//     so the softmax weights never leave registers; the only cross-lane traffic is a 2-step
//     reduction of the running maximum when it grows, and of the sum at the end.
// Online softmax keeps a reference maximum per head in log2 units; it is raised only when a page
// exceeds it by more than kRaise (any reference gives the same quotient, the bound only guards
// the fp32 range), which removes the accumulator rescale from almost every page.
#pragma once
#include <type_traits>

#include "ts_device.h"

namespace ts {

constexpr float kRaise = 16.0f;   // log2 units: weights stay below 2^16 relative to the reference

// One (page, KV head) tile in registers, D = head dim (64 or 128): K as 1 KB runs, V as 16-dim blocks.
template <typename KT, int D> struct KVTile;
template <int D> struct KVTile<uint16_t, D> { uint4 k[D / 32]; uint2 v[D / 16]; };
template <int D> struct KVTile<uint8_t, D>  { uint4 k[D / 64]; uint32_t v[D / 16]; };

// Tiles are read with the non-temporal hint: the scan touches every byte once, and keeping it out
// of the L2's replacement traffic raised the rate from 5.9 to 6.45 TB/s (bf16; fp8: 5.9 to 6.3).
template <int D>
__device__ __forceinline__ void load_tile(KVTile<uint16_t, D>& t, const char* kc, const char* vc,
                                          int64_t tile, int lane)
{
    const char* kt = kc + tile * (32 * D) + lane * 16;
    const char* vt = vc + tile * (32 * D) + (lane & 15) * 32 + (lane >> 4) * 8;
#pragma unroll
    for (int b = 0; b < D / 32; ++b) t.k[b] = load_nt4(kt + b * 1024);
#pragma unroll
    for (int b = 0; b < D / 16; ++b) t.v[b] = load_nt2(vt + b * 512);
}

template <int D>
__device__ __forceinline__ void load_tile(KVTile<uint8_t, D>& t, const char* kc, const char* vc,
                                          int64_t tile, int lane)
{
    const char* kt = kc + tile * (16 * D) + lane * 16;
    const char* vt = vc + tile * (16 * D) + (lane & 15) * 16 + (lane >> 4) * 4;
#pragma unroll
    for (int b = 0; b < D / 64; ++b) t.k[b] = load_nt4(kt + b * 1024);
#pragma unroll
    for (int b = 0; b < D / 16; ++b) t.v[b] = __builtin_nontemporal_load((const uint32_t*)(vt + b * 256));
}

// The same through buffer descriptors of the tile.  With `in` false they have no bytes, and the loads return zeros
// without touching memory: a prefetch past the end of an item keeps the number of loads in flight static and
// costs no bandwidth.  (Takes about six vector registers more than the form above, which the lean kernel lacks.)
constexpr int kRawBuffer = 0x00027000;                     // untyped 32-bit data, offsets in bytes
constexpr int kNonTemporal = 2;                            // cache policy bit
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_buffer(const char* p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, bytes, kRawBuffer);
}
template <int D>
__device__ __forceinline__ void load_tile_if(KVTile<uint16_t, D>& t, const char* kc, const char* vc,
                                             int64_t tile, int lane, bool in)
{
    const int bytes = in ? 32 * D : 0;
    const auto kr = tile_buffer(kc + tile * (32 * D), bytes), vr = tile_buffer(vc + tile * (32 * D), bytes);
    const int ko = lane * 16, vo = (lane & 15) * 32 + (lane >> 4) * 8;
#pragma unroll
    for (int b = 0; b < D / 32; ++b)
        t.k[b] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(kr, ko + b * 1024, 0, kNonTemporal));
#pragma unroll
    for (int b = 0; b < D / 16; ++b)
        t.v[b] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(vr, vo + b * 512, 0, kNonTemporal));
}
template <int D>
__device__ __forceinline__ void load_tile_if(KVTile<uint8_t, D>& t, const char* kc, const char* vc,
                                             int64_t tile, int lane, bool in)
{
    const int bytes = in ? 16 * D : 0;
    const auto kr = tile_buffer(kc + tile * (16 * D), bytes), vr = tile_buffer(vc + tile * (16 * D), bytes);
    const int ko = lane * 16, vo = (lane & 15) * 16 + (lane >> 4) * 4;
#pragma unroll
    for (int b = 0; b < D / 64; ++b)
        t.k[b] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(kr, ko + b * 1024, 0, kNonTemporal));
#pragma unroll
    for (int b = 0; b < D / 16; ++b) t.v[b] = __builtin_amdgcn_raw_buffer_load_b32(vr, vo + b * 256, 0, kNonTemporal);
}

// four e4m3 bytes -> four bf16 (exact: every e4m3 value is a bf16 value): one packed conversion per pair
__device__ __forceinline__ uint2 fp8x4_to_bf16x4(uint32_t w)
{
    uint2 r;
    r.x = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false));
    r.y = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true));
    return r;
}

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ s16x4 as_s16x4(uint2 v) { return __builtin_bit_cast(s16x4, v); }

// S^T (16 tokens x 16 columns) = K tile x Q^T for one page
template <int D>
__device__ __forceinline__ f32x4 qk_tile(const KVTile<uint16_t, D>& t, const bf16x8* qb)
{
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < D / 32; ++b)
        s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(t.k[b]), qb[b], s, 0, 0, 0);
    return s;
}
template <int D>
__device__ __forceinline__ f32x4 qk_tile(const KVTile<uint8_t, D>& t, const bf16x8* qb)
{
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < D / 64; ++j) {
        const uint2 a0 = fp8x4_to_bf16x4(t.k[j].x), a1 = fp8x4_to_bf16x4(t.k[j].y);
        const uint2 a2 = fp8x4_to_bf16x4(t.k[j].z), a3 = fp8x4_to_bf16x4(t.k[j].w);
        s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(make_uint4(a0.x, a0.y, a1.x, a1.y)),
                                                    qb[2 * j], s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(make_uint4(a2.x, a2.y, a3.x, a3.y)),
                                                    qb[2 * j + 1], s, 0, 0, 0);
    }
    return s;
}

template <int D> __device__ __forceinline__ uint2 v_operand(const KVTile<uint16_t, D>& t, int b) { return t.v[b]; }
template <int D> __device__ __forceinline__ uint2 v_operand(const KVTile<uint8_t, D>& t, int b) { return fp8x4_to_bf16x4(t.v[b]); }

// dims held by k-block b of the Q operand for lane group r (must mirror the K tile order)
template <typename KT> __device__ __forceinline__ int q_dim0(int b, int r)
{
    if constexpr (sizeof(KT) == 2) return 8 * (4 * b + r);
    else return 16 * (4 * (b >> 1) + r) + 8 * (b & 1);
}

// One workgroup of kDecWaves waves per item = (decode row, KV head, page range).  Wave w streams the
// pages begin+w, begin+w+kDecWaves, ... so the waves read neighbouring tiles at the same time; at
// the end their (max, sum, O) states meet in LDS and all threads add them up, in wave order.  A row that
// fits one item is finished here (no partial ever goes to HBM: stores into the middle of a saturated
// read stream were measured to cost ~10x their byte share); only rows longer than one workgroup's
// fair share are cut into several items whose partials go through combine_kernel.
constexpr int kDecWaves = 4;               // stand-alone decode kernel; the mixed kernel uses 8

// LDS image of the waves' states: the group's heads (at most HEADS) only, four dims of a head per entry, a row of which is
// one entry longer than the head so that the heads lie in different banks.  All threads of the workgroup add up an
// entry each.  (One wave adding up whole accumulators, unused columns included, while the others had nothing to do, was a
// serial end to every item: eight rows of 500-2500 tokens 15.3 -> 14.8 us a pass, three e4m3 rows of 30-131 Ki 92.0 -> 90.8.)
template <int WAVES, int D = 128, int HEADS = 16>
struct DecMerge {
    static constexpr int kHeads = HEADS;
    f32x4 o[WAVES][HEADS][D / 4 + 1];
    float m[WAVES][HEADS];
    float l[WAVES][HEADS];
};

// Partial results of consecutive splits of a row.  Plain form: read or written across a launch boundary.
struct SplitParts {
    float* o; float* ml; int Hq, D;
    __device__ __forceinline__ SplitParts(const AttnArgs& a, int first, int)
        : o(a.part_o + (int64_t)first * a.geo.Hq * a.geo.D), ml(a.part_ml + (int64_t)first * a.geo.Hq * 2), Hq(a.geo.Hq), D(a.geo.D) {}
    __device__ __forceinline__ void store_o(int k, int h, int d, f32x4 v) const { *(f32x4*)(o + ((int64_t)k * Hq + h) * D + d) = v; }
    __device__ __forceinline__ void store_ml(int k, int h, f32x2 v) const { *(f32x2*)(ml + ((int64_t)k * Hq + h) * 2) = v; }
    __device__ __forceinline__ f32x4 load_o(int k, int h, int d) const { return *(const f32x4*)(o + ((int64_t)k * Hq + h) * D + d); }
    __device__ __forceinline__ f32x2 load_ml(int k, int h) const { return *(const f32x2*)(ml + ((int64_t)k * Hq + h) * 2); }
};
// The same for partials that pass from one workgroup to another within a launch, perhaps between dies, whose L2
// caches do not see each other's lines: stores and loads carry the device-scope bit (sc1), which takes them past
// the L2.  (Plain stores and a device-scope release instead write back the whole L2 of the die for every item: 8
// rows of 1500 tokens then took 27.7 us a pass where the merge by a launch took 19.6.)  Byte offsets are 32 bits wide:
// n * Hq * D * 4 stays below 2^31.
struct SplitPartsThrough {
    static constexpr int kDevice = 16;                     // cache policy bit sc1
    __amdgpu_buffer_rsrc_t o, ml; int Hq, D;
    __device__ __forceinline__ SplitPartsThrough(const AttnArgs& a, int first, int n) : Hq(a.geo.Hq), D(a.geo.D)
    {
        o = __builtin_amdgcn_make_buffer_rsrc((void*)(a.part_o + (int64_t)first * Hq * D), (short)0, n * Hq * D * 4, kRawBuffer);
        ml = __builtin_amdgcn_make_buffer_rsrc((void*)(a.part_ml + (int64_t)first * Hq * 2), (short)0, n * Hq * 8, kRawBuffer);
    }
    __device__ __forceinline__ void store_o(int k, int h, int d, f32x4 v) const
    { __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), o, ((k * Hq + h) * D + d) * 4, 0, kDevice); }
    __device__ __forceinline__ void store_ml(int k, int h, f32x2 v) const
    { __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), ml, (k * Hq + h) * 8, 0, kDevice); }
    __device__ __forceinline__ f32x4 load_o(int k, int h, int d) const
    { return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(o, ((k * Hq + h) * D + d) * 4, 0, kDevice)); }
    __device__ __forceinline__ f32x2 load_ml(int k, int h) const
    { return __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(ml, (k * Hq + h) * 8, 0, kDevice)); }
};

// Merge of a row's splits, four dims of a head per thread:  out = sum o_i 2^(m_i - M) / sum l_i 2^(m_i - M).
// The splits are taken in chunks of eight, whose loads wait together; a chunk is summed relative to its own
// maximum and the chunks are added in order.  Whoever adds up a row -- its last item, or the merge launch with
// several chunks at a time -- thus rounds alike.
constexpr int kMergeChunk = 8;
struct SplitSum {
    float m = -INFINITY, l = 0.0f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    __device__ __forceinline__ void add(const SplitSum& c)
    {
        const float mn = fmaxf(m, c.m);                    // (finite: every split of a row has a key of every head)
        const float w0 = __builtin_amdgcn_exp2f(m - mn), w1 = __builtin_amdgcn_exp2f(c.m - mn);
        l = l * w0 + c.l * w1;
        o = o * w0 + c.o * w1;
        m = mn;
    }
};
struct ChunkLoads { f32x2 ml[kMergeChunk]; f32x4 o[kMergeChunk]; };
template <typename PARTS>
__device__ __forceinline__ ChunkLoads load_chunk(const PARTS& parts, int k0, int n_split, int h, int d)
{
    ChunkLoads c;
#pragma unroll
    for (int j = 0; j < kMergeChunk; ++j) c.ml[j] = parts.load_ml(min(k0 + j, n_split - 1), h);
#pragma unroll
    for (int j = 0; j < kMergeChunk; ++j) c.o[j] = parts.load_o(min(k0 + j, n_split - 1), h, d);
    return c;
}
__device__ __forceinline__ SplitSum sum_chunk(const ChunkLoads& l, int k0, int n_split)
{
    SplitSum c;
#pragma unroll
    for (int j = 0; j < kMergeChunk; ++j) c.m = fmaxf(c.m, l.ml[j].x);
#pragma unroll
    for (int j = 0; j < kMergeChunk; ++j) {
        if (k0 + j < n_split) {                            // (past the end: no weight of 0, which an infinite sum would turn into NaN)
            const float w = __builtin_amdgcn_exp2f(l.ml[j].x - c.m);
            c.l += l.ml[j].y * w;
            c.o += l.o[j] * w;
        }
    }
    return c;
}
__device__ __forceinline__ void store_merged(const AttnArgs& a, const SplitSum& s, int row, int h, int d)
{
    const float inv = (a.geo.kv_dtype == TS_FP8_E4M3 ? a.v_scale[h / a.geo.G] : 1.0f) / s.l;
    const int64_t at = ((int64_t)row * a.geo.Hq + h) * a.geo.D + d;
    if (a.geo.q_dtype == TS_F32) {
        *(f32x4_u*)((float*)a.out + at) = s.o * inv;
    } else {
        *(u32x2_u*)((uint16_t*)a.out + at) = u32x2{
            __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{s.o[0] * inv, s.o[1] * inv}, bf16x2)),
            __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{s.o[2] * inv, s.o[3] * inv}, bf16x2))};
    }
}

// An item of the device work list, through the scalar cache.
__device__ __forceinline__ DecItem load_dec_item(const DecItem* p)
{
    const int32_t TS_CONSTANT* w = as_constant((const int32_t*)p);
    return DecItem{w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7]};
}

// Two pages of a KV head in registers, taken through the softmax together (decode_pairs): K of each page, V with the two
// pages' pieces side by side, as the 16x16x32 MFMA takes its 32 tokens.
template <typename KT, int D> struct KVPair;
template <int D> struct KVPair<uint16_t, D> { uint4 k[2][D / 32]; uint4 v[D / 16]; };
template <int D> struct KVPair<uint8_t, D>  { uint4 k[2][D / 64]; uint2 v[D / 16]; };

__device__ __forceinline__ uint4 flip_signs(uint4 v)
{
    return make_uint4(v.x ^ 0x80008000u, v.y ^ 0x80008000u, v.z ^ 0x80008000u, v.w ^ 0x80008000u);
}

// (through buffer descriptors of the tile: the base is in scalar registers, and one offset register serves all loads)
template <int H, typename KT, int D>
__device__ __forceinline__ void load_pair_k(KVPair<KT, D>& t, const char* kc, int64_t tile, int ko)
{
    constexpr int kBytes = 16 * D * (int)sizeof(KT);
    const auto kr = tile_buffer(kc + tile * kBytes, kBytes);
#pragma unroll
    for (int b = 0; b < kBytes / 1024; ++b)
        t.k[H][b] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(kr, ko, b * 1024, kNonTemporal));
}
template <int H, typename KT, int D>
__device__ __forceinline__ void load_pair_v(KVPair<KT, D>& t, const char* vc, int64_t tile, int vo)
{
    constexpr int kBytes = 16 * D * (int)sizeof(KT);
    const auto vr = tile_buffer(vc + tile * kBytes, kBytes);
#pragma unroll
    for (int b = 0; b < D / 16; ++b) {
        if constexpr (sizeof(KT) == 2) {
            const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(vr, vo, b * 512, kNonTemporal);
            if constexpr (H == 0) { t.v[b].x = x.x; t.v[b].y = x.y; } else { t.v[b].z = x.x; t.v[b].w = x.y; }
        } else {
            const uint32_t x = __builtin_amdgcn_raw_buffer_load_b32(vr, vo, b * 256, kNonTemporal);
            if constexpr (H == 0) t.v[b].x = x; else t.v[b].y = x;
        }
    }
}
__device__ __forceinline__ uint32_t swap_halves16(uint32_t x)  // lanes n and n ^ 8 of every sixteen trade places
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x128, 0xf, 0xf, true);   // row rotated by 8
}

// The scan of a wave's np pages (ids at bt[step * k], k = 0 .. np - 1, the first of them page `first` of the sequence),
// two pages at a time, for groups of at most eight query heads.  Columns n and n + 8 of the score products are the same
// head (column n is head n % 8), so of the two pages' scores the lanes of columns 0-7 take the first page's and those of
// columns 8-15 the second's: one round of softmax arithmetic serves both pages.  The packed weights then trade places
// between the two halves, every column has both pages', and one 16x16x32 MFMA per 16 dims takes the 32 tokens.  Against
// a page at a time a launch has 20.6 vector instructions per page, start and merge included, for 24.4 (17.5 in the loop; e4m3, where 32
// are conversions, 52.2 for 58.5) and 8 MFMAs for 12; its loads take more
// issue cycles (V in 8-byte pieces of two tiles).  The scan alone does not notice (it waits for memory); next to prefill tiles,
// which leave it little of the vector ALU and of the matrix pipe, it counts.
// A wave's last page (the only one that can be partly filled) goes through the masked single step.
template <typename KT, int D>
__device__ __forceinline__ void decode_pairs(const AttnArgs& a, const bf16x8 (&qb)[D / 32], float c, int n_keys, int first, int step, int np,
                                             const int32_t TS_CONSTANT* bt, int g, int lane, f32x4 (&acc)[D / 16], float& m_ref, float& l)
{
    constexpr int DB = D / 16;
    const int Hkv = a.geo.Hkv, r = lane >> 4, n = lane & 15;
    const bool second = n >= 8;
    const char* kc = (const char*)a.k_cache;
    const char* vc = (const char*)a.v_cache;
    KVPair<KT, D> t;
    const int ko = lane * 16, vo = ((lane & 15) * (16 * (int)sizeof(KT)) + (lane >> 4) * (4 * (int)sizeof(KT)));
    auto page_at = [&](int k) { return bt[step * min(k, np - 1)]; };   // (past the end: the last page again)
    auto k_of = [&](int h) {
        KVTile<KT, D> x;
#pragma unroll
        for (int b = 0; b < (int)(sizeof(x.k) / sizeof(uint4)); ++b) x.k[b] = t.k[h][b];
        return x;
    };
    auto raise_if = [&](float lmax, bool both) {               // lmax: highest score of the lane's four tokens
        if (__any(lmax > m_ref + kRaise)) {                    // rare
            float full = pair32_max(pair16_max(lmax));
            if (both) full = fmaxf(full, __uint_as_float(swap_halves16(__float_as_uint(full))));
            const float m_new = fmaxf(m_ref, full);
            const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new);
#pragma unroll
            for (int b = 0; b < DB; ++b) acc[b] *= alpha;
            l *= alpha;
            m_ref = m_new;
        }
    };
    auto pack = [](float x, float y) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2)); };
    int32_t id0 = page_at(0), id1 = page_at(1);
    int32_t next0 = page_at(2), next1 = page_at(3);
    load_pair_k<0>(t, kc, (int64_t)id0 * Hkv + g, ko);
    load_pair_k<1>(t, kc, (int64_t)id1 * Hkv + g, ko);
    load_pair_v<0>(t, vc, (int64_t)id0 * Hkv + g, vo);
    load_pair_v<1>(t, vc, (int64_t)id1 * Hkv + g, vo);
    // (an opaque copy: the ids of the next pair are then read a round ahead, not where they are used)
    id0 = opaque_uniform(next0); id1 = opaque_uniform(next1);
    const bool has_tail = (first + step * (np - 1) + 1) * kPage > n_keys;   // wave-uniform
    const int n_pair = (np - (has_tail ? 1 : 0)) / 2;
    for (int p = 0; p < n_pair; ++p) {
        const f32x4 s0 = qk_tile(k_of(0), qb), s1 = qk_tile(k_of(1), qb);
        float x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = second ? s1[i] : s0[i];
        __builtin_amdgcn_sched_barrier(0);                     // (the next pages' pieces land in the registers just read)
        load_pair_k<0>(t, kc, (int64_t)id0 * Hkv + g, ko);
        load_pair_k<1>(t, kc, (int64_t)id1 * Hkv + g, ko);
        next0 = page_at(2 * p + 4); next1 = page_at(2 * p + 5);
        raise_if(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])) * c, true);
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[i], c, -m_ref));
        l += (x[0] + x[1]) + (x[2] + x[3]);
        const uint32_t w0 = pack(x[0], x[1]), w1 = pack(x[2], x[3]);
        const uint32_t o0 = swap_halves16(w0), o1 = swap_halves16(w1);
        const bf16x8 pv = as_bf16x8(make_uint4(second ? o0 : w0, second ? o1 : w1, second ? w0 : o0, second ? w1 : o1));
#pragma unroll
        for (int b = 0; b < DB; ++b) {
            uint4 vv;
            if constexpr (sizeof(KT) == 2) vv = t.v[b];
            else {
                const uint2 v0 = fp8x4_to_bf16x4(t.v[b].x), v1 = fp8x4_to_bf16x4(t.v[b].y);
                vv = make_uint4(v0.x, v0.y, v1.x, v1.y);
            }
            acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vv), pv, acc[b], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        load_pair_v<0>(t, vc, (int64_t)id0 * Hkv + g, vo);
        load_pair_v<1>(t, vc, (int64_t)id1 * Hkv + g, vo);
        id0 = next0; id1 = next1;
    }
    // the one or two pages that are left sit in t: singly, the last one with its mask
    auto single = [&](int page, auto masked) {
        constexpr bool MASKED = decltype(masked)::value;
        const f32x4 s = qk_tile(k_of(0), qb);
        const int nvalid = n_keys - (page * kPage + 4 * r);    // tokens 4 r .. 4 r + 3 valid if < nvalid
        float x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = MASKED && nvalid <= i ? -INFINITY : s[i] * c;
        raise_if(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), false);
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = __builtin_amdgcn_exp2f(x[i] - m_ref);
        l += second ? 0.0f : (x[0] + x[1]) + (x[2] + x[3]);    // (the two halves' sums are added at the end)
        const s16x4 pv = as_s16x4(make_uint2(pack(x[0], x[1]), pack(x[2], x[3])));
        const uint64_t keep = !MASKED || nvalid >= 4 ? ~0ull : (nvalid <= 0 ? 0ull : ((1ull << (16 * nvalid)) - 1ull));
#pragma unroll
        for (int b = 0; b < DB; ++b) {
            uint2 vv;
            if constexpr (sizeof(KT) == 2) vv = make_uint2(t.v[b].x, t.v[b].y); else vv = fp8x4_to_bf16x4(t.v[b].x);
            vv.x &= (uint32_t)keep; vv.y &= (uint32_t)(keep >> 32);
            acc[b] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as_s16x4(vv), pv, acc[b], 0, 0, 0);
        }
    };
    int k = 2 * n_pair;
    if (np - k == 2) {                                         // wave-uniform, as the next
        single(first + step * k, std::false_type{});
#pragma unroll
        for (int b = 0; b < (int)(sizeof(t.k[0]) / sizeof(uint4)); ++b) t.k[0][b] = t.k[1][b];
#pragma unroll
        for (int b = 0; b < DB; ++b) {
            if constexpr (sizeof(KT) == 2) { t.v[b].x = t.v[b].z; t.v[b].y = t.v[b].w; } else t.v[b].x = t.v[b].y;
        }
        ++k;
    }
    if (k < np) single(first + step * k, std::true_type{});
    l += __uint_as_float(swap_halves16(__float_as_uint(l)));
}

// One decode item for KV head g, executed by a workgroup of WAVES waves.  All waves must call it and all merge.  It contains
// one workgroup barrier per turn of HEADS heads, between the waves' writes of mg and everybody's reads, and one between two turns
// (HEADS < 16 and G > HEADS: two turns, three barriers; G is the same for all).  Nothing follows the last reads, so a barrier must come before
// mg is written again: the caller's, or (mg_busy) one in here just before the first write, so that a wave that has merged its
// share starts on the next item's pages.
// EXACT: prefetches past the end read nothing (load_tile_if).
// THROUGH: partial results of split rows are stored for arrive_and_merge.
// FUSED: the row's new token comes from a.k_new / a.v_new and is written into the cache here (see AttnArgs).
// PAIRS: at most eight query heads per KV head, two pages at a time (decode_pairs).
template <typename KT, int NBUF, int WAVES, int D = 128, bool THROUGH = false, bool FUSED = false, bool EXACT = false, bool PAIRS = false, int HEADS = 16>
__device__ __forceinline__ void decode_item(const AttnArgs& a, const DecItem it, int g, DecMerge<WAVES, D, HEADS>& mg, bool mg_busy = false)
{
    constexpr int KB = D / 32, DB = D / 16;    // 32-dim steps of K Q^T, 16-dim blocks of O^T
    const int it_row = it.row, it_seq = it.seq, it_keys = it.n_keys, it_pb = it.page_begin, it_pe = it.page_end, it_part = it.part;
    // (readfirstlane tells the compiler the wave index is uniform, which keeps everything derived
    // from it -- the page-id loads above all -- on the scalar unit)
    // (an opaque copy: where the caller loops over items the lane offsets are worked out per item instead of being
    // kept across the loop)
    const int tid = opaque((int)threadIdx.x);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, r = lane >> 4, n = lane & 15;
    const int Hq = a.geo.Hq, Hkv = a.geo.Hkv, G = a.geo.G;

    // this wave's pages: it_pb + wave + WAVES * k, k = 0 .. np-1
    const int np = max(0, (it_pe - it_pb - wave + WAVES - 1) / WAVES);
    const int32_t TS_CONSTANT* bt = as_constant(a.block_table) + (int64_t)it_seq * a.geo.max_pages + it_pb + wave;

    f32x4 acc[DB];
#pragma unroll
    for (int b = 0; b < DB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_ref = -INFINITY, l = 0.0f;

    // Fused form, e4m3 cache: the conversion of the row's new token (a division and an encoding per element) is
    // shared out over the whole workgroup, one or two elements per thread, instead of being done by the sixteen
    // lanes that need the bytes; every thread writes its V byte into the cache, the codes meet in LDS, and D/16
    // threads write the K chunks.  Only the item that holds the row's last page does this (all its waves do:
    // the condition is the same for the whole workgroup).
    [[maybe_unused]] __shared__ __align__(16) uint8_t new_tok[FUSED && sizeof(KT) == 1 ? 2 * D : 16];
    if constexpr (FUSED && sizeof(KT) == 1) {
        if (it_pe * kPage >= it_keys) {
            const int slot = (it_keys - 1) & (kPage - 1);
            const int64_t tile = (int64_t)as_constant(a.block_table)[(int64_t)it_seq * a.geo.max_pages + ((it_keys - 1) >> 4)] * Hkv + g;
            uint8_t* kc_w = (uint8_t*)const_cast<void*>(a.k_cache) + tile * (16 * D);
            uint8_t* vc_w = (uint8_t*)const_cast<void*>(a.v_cache) + tile * (16 * D);
            const uint16_t* kn = (const uint16_t*)a.k_new + ((int64_t)it_row * Hkv + g) * D;
            const uint16_t* vn = (const uint16_t*)a.v_new + ((int64_t)it_row * Hkv + g) * D;
            const float ks = a.k_scale[g], vs = a.v_scale[g];
            for (int e = threadIdx.x; e < 2 * D; e += 64 * WAVES) {
                const bool is_v = e >= D;
                const int dim = is_v ? e - D : e;
                const uint32_t code = float_to_e4m3_bits(bf16_bits_to_float(is_v ? vn[dim] : kn[dim]) / (is_v ? vs : ks));
                new_tok[e] = (uint8_t)code;
                if (is_v) __builtin_nontemporal_store((uint8_t)code, vc_w + dim * 16 + slot);
            }
            __syncthreads();
            if ((int)threadIdx.x < D / 16)
                store_nt(kc_w + (threadIdx.x * 16 + slot) * 16, *(const uint4*)(new_tok + 16 * threadIdx.x));
        }
    }

    if (np > 0) {                                                 // wave-uniform
        // Q^T operand: column n is query head g*G + n; columns >= G repeat the group's last head
        // (their results are finite and never stored)
        bf16x8 qb[KB];
        {
            const uint16_t* qrow = (const uint16_t*)a.q + ((int64_t)it_row * Hq + g * G + min(PAIRS ? n & 7 : n, G - 1)) * D;
#pragma unroll
            for (int b = 0; b < KB; ++b) qb[b] = as_bf16x8(*(const uint4*)(qrow + q_dim0<KT>(b, r)));
        }
        const float kscale = (sizeof(KT) == 1) ? a.k_scale[g] : 1.0f;
        const float c = a.sm_scale * kscale * kLog2e;
        if constexpr (PAIRS) {
            static_assert(!FUSED && !EXACT, "");
            if (c < 0.0f) {                                       // (a negative K scale: the maximum is taken before the scale)
#pragma unroll
                for (int b = 0; b < KB; ++b) qb[b] = as_bf16x8(flip_signs(__builtin_bit_cast(uint4, qb[b])));
            }
            const float cu = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(fabsf(c))));   // (in a scalar register)
            decode_pairs<KT, D>(a, qb, cu, it_keys, it_pb + wave, WAVES, np, bt, g, lane, acc, m_ref, l);
        } else {
        const char* kc = (const char*)a.k_cache;
        const char* vc = (const char*)a.v_cache;

        // page ids come through the scalar cache, one fetch ahead of their use
        int next_k = 0;
        int next_id = bt[0];
        auto fetch = [&](KVTile<KT, D>& t) {
            if constexpr (EXACT) {
                // (past the end nothing is read, but a refill of the last page's own slot repeats that page)
                load_tile_if(t, kc, vc, (int64_t)next_id * Hkv + g, lane, next_k < np || next_k == np - 1 + NBUF);
                next_k += 1;
                next_id = bt[WAVES * min(next_k, np - 1)];
            } else {
                load_tile(t, kc, vc, (int64_t)next_id * Hkv + g, lane);
                next_k = min(next_k + 1, np - 1);                 // past the end: stay on the last page
                next_id = bt[WAVES * next_k];
            }
        };
        KVTile<KT, D> buf[NBUF];
#pragma unroll
        for (int j = 0; j < NBUF; ++j) fetch(buf[j]);

        // (the wave's last page is partly filled only if it is the row's last page)
        const int page_last = it_pb + wave + WAVES * (np - 1);
        // (fused form: the row's last page always goes through the masked step, which patches in the new token)
        const bool has_tail = FUSED ? (page_last + 1) * kPage >= it_keys : (page_last + 1) * kPage > it_keys;   // wave-uniform
        const int np_main = np - (has_tail ? 1 : 0);
        // Fused form: the new token's K and V in cache form (converted exactly as the append kernels convert
        // them), asked for now so that the reads are under way during the scan.  K: the lanes of the token's slot
        // hold its dims in tile order; V: the lanes of the slot's group of four hold one element per dim block.
        constexpr int KR = sizeof(KT) == 2 ? D / 32 : D / 64;
        [[maybe_unused]] const int new_slot = (it_keys - 1) & (kPage - 1);
        [[maybe_unused]] uint4 new_k[KR];
        [[maybe_unused]] uint32_t new_v[DB];
        if constexpr (FUSED) {
            if (has_tail) {
                const uint16_t* kn = (const uint16_t*)a.k_new + ((int64_t)it_row * Hkv + g) * D;
                const uint16_t* vn = (const uint16_t*)a.v_new + ((int64_t)it_row * Hkv + g) * D;
                if constexpr (sizeof(KT) == 2) {
#pragma unroll
                    for (int b = 0; b < KR; ++b) new_k[b] = *(const uint4*)(kn + 8 * (4 * b + r));
#pragma unroll
                    for (int b = 0; b < DB; ++b) new_v[b] = vn[16 * b + n];
                } else {
                    // (converted by the whole workgroup above)
#pragma unroll
                    for (int j = 0; j < KR; ++j) new_k[j] = *(const uint4*)(new_tok + 16 * (4 * j + r));
#pragma unroll
                    for (int b = 0; b < DB; ++b) new_v[b] = new_tok[D + 16 * b + n];
                }
            }
        }

        // One page: S^T, online softmax against the reference maximum, O^T += V^T P^T.  MASKED is the row's last,
        // partly filled page: scores and V of the slots past n_keys are masked (the slots hold whatever was there
        // before).  It runs once per row, after the loop, so that the loop carries no mask arithmetic.
        auto page_step = [&](const KVTile<KT, D>& t_in, const int page, auto masked) {
            constexpr bool MASKED = decltype(masked)::value;
            KVTile<KT, D> t = t_in;
            if constexpr (MASKED && FUSED) {
                // The row's last page: slot (n_keys - 1) % 16 belongs to the token this pass appends.  Its K and V
                // (asked for before the scan, already in cache form) replace what the cache held in that slot and,
                // with a bf16 cache, go from here into the cache (an e4m3 cache got them from the workgroup above).
                const int64_t tile = (int64_t)bt[WAVES * (np - 1)] * Hkv + g;
                char* kc_w = (char*)const_cast<void*>(a.k_cache) + tile * (16 * D * (int)sizeof(KT));
                char* vc_w = (char*)const_cast<void*>(a.v_cache) + tile * (16 * D * (int)sizeof(KT));
                if (n == new_slot) {
#pragma unroll
                    for (int b = 0; b < KR; ++b) {
                        t.k[b] = new_k[b];
                        if constexpr (sizeof(KT) == 2) store_nt(kc_w + lane * 16 + b * 1024, new_k[b]);
                    }
                }
                if (r == (new_slot >> 2)) {
#pragma unroll
                    for (int b = 0; b < DB; ++b) {
                        if constexpr (sizeof(KT) == 2) {
                            const int sh = 16 * (new_slot & 1);
                            uint32_t& w = (new_slot & 2) ? t.v[b].y : t.v[b].x;
                            w = (w & ~(0xffffu << sh)) | (new_v[b] << sh);
                            __builtin_nontemporal_store((uint16_t)new_v[b], (uint16_t*)(vc_w + (16 * b + n) * 32 + new_slot * 2));
                        } else {
                            const int sh = 8 * (new_slot & 3);
                            t.v[b] = (t.v[b] & ~(0xffu << sh)) | (new_v[b] << sh);
                        }
                    }
                }
            }
            f32x4 s = qk_tile(t, qb);
            float t0 = s[0] * c, t1 = s[1] * c, t2 = s[2] * c, t3 = s[3] * c;
            const int nvalid = it_keys - (page * kPage + 4 * r);   // tokens tok0 .. tok0+3 valid if < nvalid
            if constexpr (MASKED) {
                t0 = nvalid > 0 ? t0 : -INFINITY; t1 = nvalid > 1 ? t1 : -INFINITY;
                t2 = nvalid > 2 ? t2 : -INFINITY; t3 = nvalid > 3 ? t3 : -INFINITY;
            }
            const float lmax = fmaxf(fmaxf(t0, t1), fmaxf(t2, t3));
            if (__any(lmax > m_ref + kRaise)) {           // raise the reference (rare)
                float full = fmaxf(lmax, __shfl_xor(lmax, 16, 64));
                full = fmaxf(full, __shfl_xor(full, 32, 64));
                const float m_new = fmaxf(m_ref, full);
                const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new);   // 0 on the first page
#pragma unroll
                for (int b = 0; b < DB; ++b) acc[b] *= alpha;
                l *= alpha;
                m_ref = m_new;
            }
            const float p0 = __builtin_amdgcn_exp2f(t0 - m_ref), p1 = __builtin_amdgcn_exp2f(t1 - m_ref);
            const float p2 = __builtin_amdgcn_exp2f(t2 - m_ref), p3 = __builtin_amdgcn_exp2f(t3 - m_ref);
            l += (p0 + p1) + (p2 + p3);
            uint2 pw;
            pw.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{p0, p1}, bf16x2));
            pw.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{p2, p3}, bf16x2));
            const s16x4 pv = as_s16x4(pw);
            uint64_t keep = ~0ull;
            if constexpr (MASKED) keep = nvalid >= 4 ? ~0ull : (nvalid <= 0 ? 0ull : ((1ull << (16 * nvalid)) - 1ull));
#pragma unroll
            for (int b = 0; b < DB; ++b) {
                uint2 vv = v_operand(t, b);
                if constexpr (MASKED) { vv.x &= (uint32_t)keep; vv.y &= (uint32_t)(keep >> 32); }
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as_s16x4(vv), pv, acc[b], 0, 0, 0);
            }
        };
        for (int base = 0; base < np_main; base += NBUF) {
#pragma unroll
            for (int j = 0; j < NBUF; ++j) {
                const int k = base + j;
                if (k < np_main) page_step(buf[j], it_pb + wave + WAVES * k, std::false_type{});   // wave-uniform
                fetch(buf[j]);                                    // refill
            }
        }
        if (has_tail) {
            const int jt = (np - 1) % NBUF;                       // the last page's slot
#pragma unroll
            for (int j = 0; j < NBUF; ++j)
                if (j == jt) page_step(buf[j], page_last, std::true_type{});
        }
        }
    }

    float l_tot = l + __shfl_xor(l, 16, 64);
    l_tot += __shfl_xor(l_tot, 32, 64);

    const int tid_o = opaque((int)threadIdx.x), lane_o = tid_o & 63, r_o = lane_o >> 4, n_o = lane_o & 15;   // (derived afresh: see above)
    // ---- merge the waves' states (wave order, so the result is reproducible) ----------------------
    if (mg_busy) __syncthreads();
    const float vscale = (sizeof(KT) == 1) ? a.v_scale[g] : 1.0f;
    int h0 = 0;                                                   // (groups of more heads than the image holds: in turns)
    do {
        if (n_o >= h0 && n_o < min(G, h0 + HEADS)) {
#pragma unroll
            for (int b = 0; b < DB; ++b) mg.o[wave][n_o - h0][4 * b + r_o] = acc[b];
            if (r_o == 0) { mg.m[wave][n_o - h0] = m_ref; mg.l[wave][n_o - h0] = l_tot; }
        }
        __syncthreads();
        for (int i = tid_o; i < min(G - h0, HEADS) * (D / 4); i += 64 * WAVES) {
            const int hd = i / (D / 4), dq = i % (D / 4), h = g * G + h0 + hd;
            float M = mg.m[0][hd];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) M = fmaxf(M, mg.m[w][hd]);
            // wave 0 always holds the item's first page, so M is finite; exp2(-inf) = 0 for a wave without pages
            const float w0 = __builtin_amdgcn_exp2f(mg.m[0][hd] - M);
            f32x4 o = mg.o[0][hd][dq] * w0;
            float lsum = mg.l[0][hd] * w0;
#pragma unroll
            for (int w = 1; w < WAVES; ++w) {
                const float ww = __builtin_amdgcn_exp2f(mg.m[w][hd] - M);
                lsum += mg.l[w][hd] * ww;
                o += mg.o[w][hd][dq] * ww;
            }
            if (it_part < 0) {
                const float inv = vscale / lsum;
                uint2 w;
                w.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{o[0] * inv, o[1] * inv}, bf16x2));
                w.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{o[2] * inv, o[3] * inv}, bf16x2));
                *(uint2*)((uint16_t*)a.out + ((int64_t)it_row * Hq + h) * D + 4 * dq) = w;
            } else {
                const std::conditional_t<THROUGH, SplitPartsThrough, SplitParts> parts(a, it_part, 1);
                parts.store_o(0, h, 4 * dq, o);
                if (dq == 0) parts.store_ml(0, h, f32x2{M, lsum});
            }
        }
        h0 += HEADS;
        if (HEADS < 16 && h0 < G) __syncthreads();
    } while (HEADS < 16 && h0 < G);
}

// The end of a workgroup whose items [first, first + n) held parts of split rows: the last item of a row to get here
// merges the row's partials (no launch for the merge).  The partials were stored past the die's L2 (see
// SplitPartsThrough), so once the stores are acknowledged they are where every other workgroup's loads of the same
// kind find them; only then is the arrival counted.  Whoever counts a row's last arrival reads all its partials
// back, its own included, in split order: the result does not depend on which item came last.  One wait and one
// round of counting serve all items of the workgroup (n <= 64).  All threads call it.
// TWO: two chunks of splits at a time (more registers, so in the form of few rows only: its last workgroup's reads are
// the end of the pass).
template <int D, int THREADS, bool TWO>
__device__ __forceinline__ void arrive_and_merge(const AttnArgs& a, const DecItem* items, int n, const CmbItem* rows, int g)
{
    __shared__ uint64_t s_last;
    const int tid = threadIdx.x;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // each wave waits for its own stores, the barrier for all
    __syncthreads();
    if (tid < 64) {
        bool last = false;
        const int row = tid < n ? items[tid].cmb : -1;
        if (row >= 0) {
            int32_t* ctr = a.cmb_ctr + (int64_t)row * a.geo.Hkv + g;
            const int n_split = rows[row].n_split;
            last = __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_split - 1;
            if (last) __hip_atomic_store(ctr, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next launch
        }
        const uint64_t m = __ballot(last);
        if (tid == 0) s_last = m;
    }
    __syncthreads();
    uint64_t todo = s_last;
    asm volatile("" ::: "memory");
    while (todo) {                                         // (the same for every thread)
        const int j = __builtin_ctzll(todo);
        todo &= todo - 1;
        const CmbItem row = rows[items[j].cmb];
        const SplitPartsThrough parts(a, row.part_begin, row.n_split);
        for (int i = tid; i < a.geo.G * (D / 4); i += THREADS) {
            const int h = g * a.geo.G + i / (D / 4), d = i % (D / 4) * 4;
            SplitSum sum;
            for (int k0 = 0; k0 < row.n_split; k0 += (TWO ? 2 : 1) * kMergeChunk) {
                const ChunkLoads c0 = load_chunk(parts, k0, row.n_split, h, d);
                if (TWO && k0 + kMergeChunk < row.n_split) {
                    const ChunkLoads c1 = load_chunk(parts, k0 + kMergeChunk, row.n_split, h, d);
                    sum.add(sum_chunk(c0, k0, row.n_split));
                    sum.add(sum_chunk(c1, k0 + kMergeChunk, row.n_split));
                } else {
                    sum.add(sum_chunk(c0, k0, row.n_split));
                }
            }
            store_merged(a, sum, row.row, h, d);
        }
    }
}

}  // namespace ts
