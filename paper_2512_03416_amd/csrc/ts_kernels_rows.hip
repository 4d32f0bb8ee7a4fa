// Generic row tiles: softmax attention in fp32 arithmetic throughout, any supported element type and head dim.
// They serve the fp32 configuration (where the 1e-5 bar rules out bf16 matrix instructions) and the chunk rows
// that the bf16 tiles do not take (option prefill_path; head dim 64 over an e4m3 cache too large to widen).
//
// A tile is 16 columns = (16 / G consecutive tokens of one sequence) x (G query heads of one KV head) over a range
// of cache pages; a decode row is a tile of one token (paper Sec. 2.1, Sec. 3.4: the two differ only in how many
// keys they see).  Both products run on the fp32 matrix instruction 16x16x4 -- an fp32 fused multiply-add per
// element into fp32 accumulators -- so every K/V byte that is loaded serves 16 columns:
//   - S^T = K Q^T: a lane's 16-byte piece of a K tile is X consecutive dims of one token; step e of piece b
//     multiplies dims (4 b + r) X + e of the four lane groups r.  The order of a contraction is free, and this
//     one takes the cache layout as it is;
//   - O^T += V^T P^T: the accumulator of S^T (lane (r, n): tokens 4r .. 4r+3 of column n) is the B operand of
//     step e as it stands, a lane's four tokens of a V row are the matching A operands.
// Four waves share a tile: each takes every fourth page with the next page's loads in flight, and their states
// meet in LDS.  Long tiles are cut along the pages like decode rows (merged by combine_kernel).
//
// What bounds it: chunk rows, the matrix instruction (64 flop per clock and SIMD: 2048 clocks per page and KV head
// with head dim 128); decode rows, HBM.
//
// Decode rows of groups of at most four heads (fp32) would fill four of the sixteen columns and take the matrix
// instructions' time four times over -- next to chunk tiles on the same SIMD that is what bounds the pass.  They take the
// form with sixteen blocks of 4x4x1 instead, 512 clocks per page and KV head: ROWS4 below.
#include <type_traits>

#include "ts_device.h"
#include "ts_launch.h"

namespace ts {

constexpr int kRtWaves = 4;
constexpr float kRaiseRt = 16.0f;      // log2 units a score may exceed the reference maximum by before it is raised
// Reference maximum of a column that has seen no key.  Finite, so that differences stay defined, and the lowest value of
// the type: any higher score raises it (16 is less than a step of the type there), a score equal to it has weight 1.
constexpr float kNoKey = -3.402823466e38f;

// One (page, KV head) tile in registers: D / 4 elements of K and of V per lane.
template <typename KT, int D> struct RtTile {
    static constexpr int X = 16 / (int)sizeof(KT), KB = D / (4 * X), VB = D / 16;
    using VPiece = std::conditional_t<sizeof(KT) == 4, uint4, std::conditional_t<sizeof(KT) == 2, uint2, uint32_t>>;
    uint4 k[KB];
    VPiece v[VB];
};

// in: else nothing is read (a buffer of no bytes, whose loads return zeros).  The prefetch needs no branch that way; it
// used to repeat a wave's last page up to three times: 4 rows and 2 chunks of 200-300 tokens (32/8 heads of 128, fp32)
// 59.0 -> 53.5 us a pass, 24 rows and 2 chunks with head dim 64 48.1 -> 46.1.
constexpr int kRtRaw = 0x00027000;                         // buffer of untyped 32-bit data, offsets in bytes
template <int POLICY, typename KT, int D>
__device__ __forceinline__ void rt_load_k(RtTile<KT, D>& t, const char* kc, int64_t tile, int lane, bool in)
{
    constexpr int kBytes = 16 * D * (int)sizeof(KT);
    const auto kr = __builtin_amdgcn_make_buffer_rsrc((void*)(kc + tile * kBytes), (short)0, in ? kBytes : 0, kRtRaw);
    const int ko = lane * 16;
#pragma unroll
    for (int b = 0; b < RtTile<KT, D>::KB; ++b) t.k[b] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(kr, ko + b * 1024, 0, POLICY));
}
template <int POLICY, typename KT, int D>
__device__ __forceinline__ void rt_load_v(RtTile<KT, D>& t, const char* vc, int64_t tile, int lane, bool in)
{
    using T = RtTile<KT, D>;
    constexpr int ES = (int)sizeof(KT), kBytes = 16 * D * ES;
    const auto vr = __builtin_amdgcn_make_buffer_rsrc((void*)(vc + tile * kBytes), (short)0, in ? kBytes : 0, kRtRaw);
    const int vo = (lane & 15) * (16 * ES) + (lane >> 4) * (4 * ES);
#pragma unroll
    for (int b = 0; b < T::VB; ++b) {
        const int at = vo + b * (256 * ES);
        if constexpr (ES == 4) t.v[b] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(vr, at, 0, POLICY));
        else if constexpr (ES == 2) t.v[b] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(vr, at, 0, POLICY));
        else t.v[b] = __builtin_amdgcn_raw_buffer_load_b32(vr, at, 0, POLICY);
    }
}

// element e of a register's worth of cache elements, as fp32 (exact for every type)
template <typename KT> __device__ __forceinline__ float rt_elem(uint32_t w, int e)
{
    if constexpr (sizeof(KT) == 4) return __uint_as_float(w);
    else if constexpr (sizeof(KT) == 2) return __uint_as_float(e ? w & 0xffff0000u : w << 16);
    else {
        const auto p = e < 2 ? __builtin_amdgcn_cvt_pk_f32_fp8((int)w, false) : __builtin_amdgcn_cvt_pk_f32_fp8((int)w, true);
        return p[e & 1];
    }
}
__device__ __forceinline__ uint32_t word_of(const uint4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }
__device__ __forceinline__ uint32_t word_of(const uint2& v, int i) { return i == 0 ? v.x : v.y; }
__device__ __forceinline__ uint32_t word_of(const uint32_t& v, int) { return v; }

// a lane's four tokens of a V row (e: a constant): is element e an infinity or a NaN (e4m3: S.1111.111), and a 0 in its place
template <typename KT, typename V> __device__ __forceinline__ bool rt_not_finite(const V& v, int e)
{
    constexpr int EW = 4 / (int)sizeof(KT);
    constexpr uint32_t kExp = sizeof(KT) == 4 ? 0x7f800000u : sizeof(KT) == 2 ? 0x7f80u : 0x7fu;
    const uint32_t m = kExp << (8 * (int)sizeof(KT) * (e % EW));
    return (word_of(v, e / EW) & m) == m;
}
// the same over all elements of all rows
template <typename KT, typename V, int N> __device__ __forceinline__ bool rt_any_not_finite(const V (&v)[N])
{
    if constexpr (sizeof(KT) == 4) {
        float x = 0.0f, y = 0.0f;                              // (0 as long as every value is finite: one instruction per value)
#pragma unroll
        for (int b = 0; b < N; ++b) {
            x = fmaf(__uint_as_float(v[b].x), 0.0f, x); y = fmaf(__uint_as_float(v[b].y), 0.0f, y);
            x = fmaf(__uint_as_float(v[b].z), 0.0f, x); y = fmaf(__uint_as_float(v[b].w), 0.0f, y);
        }
        return x + y != 0.0f;
    } else {
        bool x = false;
#pragma unroll
        for (int b = 0; b < N; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) x |= rt_not_finite<KT>(v[b], e);
        return x;
    }
}
template <typename KT, typename V> __device__ __forceinline__ void rt_clear_if(V& v, int e, bool clear)
{
    if constexpr (sizeof(KT) == 4) (e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w) = clear ? 0u : word_of(v, e);
    else if constexpr (sizeof(KT) == 2) (e < 2 ? v.x : v.y) &= clear ? ~(0xffffu << (16 * (e & 1))) : ~0u;
    else v &= clear ? ~(0xffu << (8 * e)) : ~0u;
}

template <int D> struct RtMerge {                          // LDS image of the non-leading waves' state
    float o[kRtWaves - 1][D / 16][64][4];
    float m[kRtWaves - 1][16];
    float l[kRtWaves - 1][16];
};

// KV heads vary fastest over the grid (as in the decode kernel: the Hkv tiles of a page are neighbours in memory,
// and with eight heads every tile of a (sequence, head) stream runs on one die, whose L2 then holds its pages).
template <typename QT, typename KT, int D>
__global__ __launch_bounds__(64 * kRtWaves, D == 64 ? 4 : 2) void row_tile_kernel(AttnArgs a)
{
    using T = RtTile<KT, D>;
    constexpr int X = T::X, KB = T::KB, VB = T::VB, EW = 4 / (int)sizeof(KT);   // EW: elements per register
    __shared__ RtMerge<D> mg;
    const int Hq = a.geo.Hq, Hkv = a.geo.Hkv, G = a.geo.G;
    const int32_t TS_CONSTANT* w = as_constant((const int32_t*)(a.rt + blockIdx.x / Hkv));
    struct { int seq, row0, pos0, n_tok, page_begin, page_end, part, n_split; } it{w[0], w[1], w[2], w[3] & 255, 0, 0, -1, 1};
    it.page_end = (it.pos0 + it.n_tok - 1) / kPage + 1;
    if (w[3] >> 8) {                                       // a range of the tile's pages
        const int32_t TS_CONSTANT* cut = as_constant((const int32_t*)(a.rtcut + ((w[3] >> 8) - 1)));
        it.page_begin = cut[0]; it.page_end = cut[1]; it.part = cut[2]; it.n_split = cut[3];
    }
    const int g = blockIdx.x % Hkv;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, r = lane >> 4, n = lane & 15;

    // column n = (token t, head g G + hd); columns past the tile's last token repeat it and are never stored
    const int t_raw = n / G, hd = n - t_raw * G;
    const int t = min(t_raw, it.n_tok - 1);
    const int keys = it.pos0 + t + 1;                      // keys this column sees
    const int keys_min = it.pos0 + 1, keys_max = it.pos0 + it.n_tok;   // over the tile's columns

    // this wave's pages: page_begin + wave + kRtWaves * k, k = 0 .. np - 1
    const int np = max(0, (it.page_end - it.page_begin - wave + kRtWaves - 1) / kRtWaves);
    const int32_t TS_CONSTANT* bt = as_constant(a.block_table) + (int64_t)it.seq * a.geo.max_pages + it.page_begin + wave;

    f32x4 acc[VB];
#pragma unroll
    for (int b = 0; b < VB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_ref = kNoKey, l = 0.0f;

    // ROWS4: one token, at most four heads.  Lane (r, n) is row n % 4 or column n % 4 of block (r, n / 4):
    //   - S^T: block (r, n / 4) multiplies tokens 4 (n / 4) .. + 3 with heads 0 .. 3 over the dims of lane group r (the K
    //     pieces as they are); the lane groups' sums are added, and every lane of column j has the scores of the four
    //     tokens of its block for head j;
    //   - O^T: block (r, n / 4) multiplies dims 16 b + 4 (n / 4) .. + 3 with the weights of tokens 4 r .. + 3 (the V pieces as
    //     they are), which lane (r, n) fetches from the block that holds them; the lane groups' sums are added at the end.
    auto scan = [&](auto rows4) {
        constexpr bool ROWS4 = decltype(rows4)::value;
        constexpr int kPolicy = ROWS4 ? 2 : 0;             // non-temporal: nobody else reads a decode row's pages
        const int from = 4 * (20 * r + (n & 3));           // lane (r, 4 r + n % 4), as a byte index
        float q[D / 4];                                    // B operands of K Q^T: dims (4 b + r) X + e of the column
        {
            const QT* qrow = (const QT*)a.q + ((int64_t)(it.row0 + t) * Hq + g * G + (ROWS4 ? min(n & 3, G - 1) : hd)) * D;
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
                for (int e = 0; e < X; ++e) {
                    const QT v = qrow[(4 * b + r) * X + e];
                    if constexpr (sizeof(QT) == 4) q[b * X + e] = v;
                    else q[b * X + e] = bf16_bits_to_float(v);
                }
        }
        const float c = a.sm_scale * (sizeof(KT) == 1 ? a.k_scale[g] : 1.0f) * kLog2e;
        const char* kc = (const char*)a.k_cache;
        const char* vc = (const char*)a.v_cache;
        int next_k = 0, next_id = bt[0];
        auto fetch = [&](T& tile) {
            rt_load_k<kPolicy, KT, D>(tile, kc, (int64_t)next_id * Hkv + g, lane, next_k < np);
            rt_load_v<kPolicy, KT, D>(tile, vc, (int64_t)next_id * Hkv + g, lane, next_k < np);
            next_k += 1;
            next_id = bt[kRtWaves * min(next_k, np - 1)];
        };
        // One page.  MASKED: it reaches past the first token's keys: scores of keys that a column does not see, and V of
        // slots that no column sees, are masked.
        // behind_k: called when K has been used.
        auto step = [&](T& tile, int page, auto masked, auto&& behind_k) {
            constexpr bool MASKED = decltype(masked)::value;
            f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;      // (two chains: half the rounding steps in a row)
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
                for (int e = 0; e < X; ++e) {
                    const float kv = rt_elem<KT>(word_of(tile.k[b], e / EW), e % EW);
                    f32x4& s = (e & 1) ? s1 : s0;
                    if constexpr (ROWS4) s = __builtin_amdgcn_mfma_f32_4x4x1f32(kv, q[b * X + e], s, 0, 0, 0);
                    else s = __builtin_amdgcn_mfma_f32_16x16x4f32(kv, q[b * X + e], s, 0, 0, 0);
                }
            float x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = (ROWS4 ? pair32_sum(pair16_sum(s0[i] + s1[i])) : s0[i] + s1[i]) * c;
            behind_k();
            const int tok0 = page * kPage + 4 * r;         // first of the lane's tokens in V ...
            const int score0 = ROWS4 ? page * kPage + (n & 12) : tok0;   // ... and of its scores
            if constexpr (MASKED) {
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i] = score0 + i < keys ? x[i] : -INFINITY;
            }
            const float lmax = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
            if (__any(lmax > m_ref + kRaiseRt)) {          // raise the reference (rare)
                float full;
                if constexpr (ROWS4) {
                    full = fmaxf(lmax, rotate16<4>(lmax));
                    full = fmaxf(full, rotate16<8>(full));
                } else {
                    full = fmaxf(lmax, __shfl_xor(lmax, 16, 64));
                    full = fmaxf(full, __shfl_xor(full, 32, 64));
                }
                const float m_new = fmaxf(m_ref, full);
                const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new);
#pragma unroll
                for (int b = 0; b < VB; ++b) acc[b] *= alpha;
                l *= alpha;
                m_ref = m_new;
            }
            float p[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(x[i] - m_ref);
            l += (p[0] + p[1]) + (p[2] + p[3]);
            if constexpr (MASKED) {                        // slots that no column sees hold whatever was there before
#pragma unroll
                for (int b = 0; b < VB; ++b)
#pragma unroll
                    for (int e = 0; e < 4; ++e) rt_clear_if<KT>(tile.v[b], e, tok0 + e >= keys_max);
                // A weight of 0 does not undo an infinite or NaN value: the columns of earlier tokens must not meet the V
                // of later ones at all.  Tokens with such a value (rare, wave-uniform) are added on the vector ALU, to
                // the columns that see them, and cleared for the product.
                if (!ROWS4 && keys_min < keys_max && __any(rt_any_not_finite<KT>(tile.v))) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        bool odd_e = false;
#pragma unroll
                        for (int b = 0; b < VB; ++b) odd_e |= rt_not_finite<KT>(tile.v[b], e);
                        uint64_t odd = __ballot(odd_e);    // lanes 16 g4 .. + 15 hold V and weights of token 4 g4 + e
                        for (int g4 = 0; odd; ++g4, odd >>= 16) {
                            if ((odd & 0xffff) == 0) continue;
                            const bool seen = page * kPage + 4 * g4 + e < keys;
                            const float w = __shfl(p[e], 16 * g4 + n, 64);
#pragma unroll
                            for (int b = 0; b < VB; ++b) {
                                const float mine = rt_elem<KT>(word_of(tile.v[b], e / EW), e % EW);
#pragma unroll
                                for (int i = 0; i < 4; ++i) {
                                    const float v = __shfl(mine, 16 * g4 + 4 * r + i, 64);
                                    acc[b][i] = fmaf(w, seen ? v : 0.0f, acc[b][i]);
                                }
                                rt_clear_if<KT>(tile.v[b], e, r == g4);
                            }
                        }
                    }
                }
            }
            if constexpr (ROWS4) {
#pragma unroll
                for (int i = 0; i < 4; ++i) p[i] = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(p[i])));
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int b = 0; b < VB; ++b) {
                    const float v = rt_elem<KT>(word_of(tile.v[b], e / EW), e % EW);
                    if constexpr (ROWS4) acc[b] = __builtin_amdgcn_mfma_f32_4x4x1f32(v, p[e], acc[b], 0, 0, 0);
                    else acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, p[e], acc[b], 0, 0, 0);
                }
        };
        // Pages past the first token's keys are the tile's last one or two (it has at most 16 tokens), so a wave has at most
        // one of them and it comes last: the loop carries no mask arithmetic, and what the masked page needs in registers
        // it finds in the buffer that is not filled any more.
        const int first = it.page_begin + wave, page_last = first + kRtWaves * (np - 1);
        const bool has_tail = (page_last + 1) * kPage > keys_min;   // wave-uniform
        const int np_main = np - (has_tail ? 1 : 0);
        if constexpr (ROWS4) {
            // One page in flight per wave, K and V of the next one asked for as soon as this one's are used, with the
            // non-temporal hint: with two pages 264 workgroups had 34 MB on the way, five microseconds of memory traffic, which
            // is slower by itself and stands in front of every load of the chunk tiles, and what they read pushed the
            // chunks' pages out of the L2.  16 rows of 64-2048 tokens next to a 231-token chunk over 300 (32/8 heads of
            // 128) 57.0 -> 51.5 us a pass, without the chunk 42.4 -> 36.5, 32 rows of 500-2048 76.3 -> 67.1.
            T t;
            fetch(t);
            for (int k = 0; k < np_main; ++k) {
                const int64_t tile = (int64_t)next_id * Hkv + g;
                const bool in = next_k < np;
                step(t, first + kRtWaves * k, std::false_type{}, [&] {
                    __builtin_amdgcn_sched_barrier(0);
                    rt_load_k<kPolicy, KT, D>(t, kc, tile, lane, in);
                    next_k += 1;
                    next_id = bt[kRtWaves * min(next_k, np - 1)];
                });
                __builtin_amdgcn_sched_barrier(0);
                rt_load_v<kPolicy, KT, D>(t, vc, tile, lane, in);
            }
            if (has_tail) step(t, page_last, std::true_type{}, [] {});
        } else {
            T buf[2];
            fetch(buf[0]);
            fetch(buf[1]);
            for (int k = 0; k < np_main; k += 2) {
                step(buf[0], first + kRtWaves * k, std::false_type{}, [] {});
                fetch(buf[0]);
                if (k + 1 >= np_main) break;               // (the second buffer may hold the masked page)
                step(buf[1], first + kRtWaves * (k + 1), std::false_type{}, [] {});
                fetch(buf[1]);
            }
            if (has_tail) {
                if ((np - 1) & 1) buf[0] = buf[1];
                step(buf[0], page_last, std::true_type{}, [] {});
            }
        }
        if constexpr (ROWS4) {                             // to the order of the other form: dims 16 b + 4 r .. + 3 of column n
#pragma unroll
            for (int b = 0; b < VB; ++b)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    acc[b][i] = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(pair32_sum(pair16_sum(acc[b][i])))));
            l += rotate16<4>(l);
            l += rotate16<8>(l);
        } else {
            l += __shfl_xor(l, 16, 64);
            l += __shfl_xor(l, 32, 64);
        }
    };
    if (np > 0) {                                          // wave-uniform
        if constexpr (sizeof(KT) == 4) {
            if (G <= 4 && it.n_tok == 1) scan(std::true_type{}); else scan(std::false_type{});
        } else {
            scan(std::false_type{});
        }
    }
    float l_tot = l;

    // merge the waves' states in wave order (results are run-to-run identical)
    if (wave > 0) {
#pragma unroll
        for (int b = 0; b < VB; ++b) *(f32x4*)mg.o[wave - 1][b][lane] = acc[b];
        if (r == 0) { mg.m[wave - 1][n] = m_ref; mg.l[wave - 1][n] = l_tot; }
    }
    __syncthreads();
    if (wave != 0) return;
    float M = m_ref;
#pragma unroll
    for (int v = 0; v < kRtWaves - 1; ++v) M = fmaxf(M, mg.m[v][n]);
    {
        const float w0 = __builtin_amdgcn_exp2f(m_ref - M);
#pragma unroll
        for (int b = 0; b < VB; ++b) acc[b] *= w0;
        l_tot *= w0;
    }
#pragma unroll
    for (int v = 0; v < kRtWaves - 1; ++v) {
        const float wv = __builtin_amdgcn_exp2f(mg.m[v][n] - M);
        l_tot += mg.l[v][n] * wv;
#pragma unroll
        for (int b = 0; b < VB; ++b) acc[b] += *(const f32x4*)mg.o[v][b][lane] * wv;
    }
    if (t_raw >= it.n_tok) return;
    const int h = g * G + hd;
    if (it.part >= 0) {                                    // a cut tile: token t's partial results are n_split slots in a row
        const int64_t slot = (int64_t)it.part + (int64_t)t * it.n_split;
        float* o = a.part_o + (slot * Hq + h) * D + 4 * r;
#pragma unroll
        for (int b = 0; b < VB; ++b) *(f32x4*)(o + 16 * b) = acc[b];
        if (r == 0) *(float2*)(a.part_ml + (slot * Hq + h) * 2) = make_float2(M, l_tot);
        return;
    }
    const float inv = (sizeof(KT) == 1 ? a.v_scale[g] : 1.0f) / l_tot;
    QT* o = (QT*)a.out + ((int64_t)(it.row0 + t) * Hq + h) * D + 4 * r;
#pragma unroll
    for (int b = 0; b < VB; ++b) {
        if constexpr (sizeof(QT) == 4) {
            *(f32x4_u*)(o + 16 * b) = acc[b] * inv;
        } else {
            *(u32x2_u*)(o + 16 * b) = u32x2{
                __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{acc[b][0] * inv, acc[b][1] * inv}, bf16x2)),
                __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{acc[b][2] * inv, acc[b][3] * inv}, bf16x2))};
        }
    }
}

template <typename QT, typename KT>
static int launch_rows_d(const AttnArgs& a, hipStream_t st, hipEvent_t done)
{
    if (a.geo.D != 64 && a.geo.D != 128) return (int)hipErrorInvalidValue;
    const int64_t most = kMaxWorkgroups > a.geo.Hkv ? kMaxWorkgroups / a.geo.Hkv : 1;
    int e = (int)hipSuccess;
    for (int64_t first = 0, left = a.n_rt; left > 0 && e == (int)hipSuccess; first += most, left -= most) {
        AttnArgs part = a;
        part.rt = a.rt + first;
        const dim3 grid((unsigned)(left < most ? left : most) * (unsigned)a.geo.Hkv), block(64 * kRtWaves);
        const hipEvent_t ev = left <= most ? done : nullptr;
        if (a.geo.D == 64) e = launch_kernel(row_tile_kernel<QT, KT, 64>, grid, block, st, ev, part);
        else e = launch_kernel(row_tile_kernel<QT, KT, 128>, grid, block, st, ev, part);
    }
    return e;
}

int launch_rows(const AttnArgs& a, void* stream, void* done)
{
    if (a.n_rt <= 0) return (int)hipSuccess;
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t ev = (hipEvent_t)done;
    if (a.geo.q_dtype == TS_F32 && a.geo.kv_dtype == TS_F32) return launch_rows_d<float, float>(a, st, ev);
    if (a.geo.q_dtype == TS_BF16 && a.geo.kv_dtype == TS_BF16) return launch_rows_d<uint16_t, uint16_t>(a, st, ev);
    if (a.geo.q_dtype == TS_BF16 && a.geo.kv_dtype == TS_FP8_E4M3) return launch_rows_d<uint16_t, uint8_t>(a, st, ev);
    return (int)hipErrorInvalidValue;
}

}  // namespace ts
