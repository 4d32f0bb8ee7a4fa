// Step a2 (+a4): launchers of the decode kernel and of the merge of split rows.
#include <algorithm>

#include "ts_decode_item.h"
#include "ts_launch.h"

namespace ts {

// KV heads vary fastest over the grid: the Hkv workgroups of one item start together and read the
// Hkv adjacent tiles of each page (one contiguous run of the cache) at about the same time.
template <typename KT, int NBUF, int D, bool EXACT, int HEADS = 16>
__device__ __forceinline__ void decode_workgroup(const AttnArgs& a)
{
    __shared__ DecMerge<kDecWaves, D, HEADS> mg;
    const int w = blockIdx.x / a.geo.Hkv, g = blockIdx.x % a.geo.Hkv;
    int first = w, end = w + 1;
    if (a.dec_wg) { first = as_constant(a.dec_wg)[w]; end = as_constant(a.dec_wg)[w + 1]; }
    bool split = false;
    for (int i = first; i < end; ++i) {
        const DecItem it = load_dec_item(a.dec + i);
        split |= it.part >= 0;
        decode_item<KT, NBUF, kDecWaves, D, true, false, EXACT>(a, it, g, mg, i > first);
    }
    if (split && a.cmb_ctr) arrive_and_merge<D, 64 * kDecWaves, false>(a, a.dec + first, end - first, a.cmb, g);
}

// (the image of eight heads, 17 KB, as in the forms below: by option this kernel runs next to resident prefill workgroups too,
// and with an e4m3 cache and three tiles it fits there, where the image of sixteen, 34 KB, made the scan wait for the tiles:
// 128 rows of 1024-8192 tokens next to 4 chunks of 2048, 64/8 heads, 1095 -> 902 us a pass.  Alone the second turn of groups of more than eight
// heads costs nothing: 20 rows of 500-8000 tokens with 128/8 heads 60.6 us either way)
template <typename KT, int NBUF, int D>
__global__ __launch_bounds__(64 * kDecWaves) void decode_kernel(AttnArgs a) { decode_workgroup<KT, NBUF, D, true, 8>(a); }

// The default forms, two KV tiles in flight per wave, held to 128 vector registers per lane (the attribute
// counts in units of two here): one such workgroup then fits on a CU next to a resident prefill workgroup
// (see prefill_resident_kernel), and four fit on a CU of their own.  A single workgroup of four waves per CU
// already keeps enough loads in flight for the bf16 scan to run at its full rate.
// decode_kernel_lean: one item per workgroup, no merge in the kernel -- next to resident prefill workgroups the
// shorter code is worth 1.5 % of the pair (the burst configuration: 633 us a pass against 643).  Head dim 128 (up to eight heads
// per KV head): two pages at a time, fewer vector and matrix instructions (see decode_pairs).  What bounds it there is not memory but what the tiles leave it
// of the SIMDs: a 4096-token chunk over 4096 next to 128 rows, a prefill workgroup on every CU, 570 -> 500 us a pass (and
// with that more of the CUs can hold one); 256 rows of 256-1500 tokens next to 2048 tokens 218 -> 210; where the tiles
// outlast the scan it changes nothing (the burst configuration, 64 Ki prompt tokens next to 512 rows).  Groups of more heads run
// decode_kernel_lean_merging there (the page-by-page scan in the short form no longer fits 128 registers since all of a
// workgroup's threads merge).
template <typename KT, int D>
__global__ __launch_bounds__(64 * kDecWaves) __attribute__((amdgpu_num_vgpr(64))) void decode_kernel_lean(AttnArgs a)
{
    __shared__ DecMerge<kDecWaves, D, 8> mg;               // (what resident prefill workgroups leave of a CU's LDS: 32 KB)
    static_assert(D == 128, "");
    decode_item<KT, 2, kDecWaves, D, false, false, false, true>(a, load_dec_item(a.dec + blockIdx.x / a.geo.Hkv), blockIdx.x % a.geo.Hkv, mg);
}
template <typename KT, int D>
__global__ __launch_bounds__(64 * kDecWaves) __attribute__((amdgpu_num_vgpr(64))) void decode_kernel_lean_merging(AttnArgs a)
{
    decode_workgroup<KT, 2, D, false, 8>(a);
}

// A launch on its own (no resident prefill workgroups next to it): prefetches past the end of an item read nothing.  A
// wave of decode_kernel_lean repeats its last page up to three times, which matters where rows are short (a wave of a
// row of 100 tokens has two pages): 200 rows of 16-200 tokens 34.4 -> 31.3 us a pass, 140 of 100-400 39.1 -> 36.3, 500
// of 100-600 152 -> 142.  (Rows of thousands of tokens, and batches of items cut or dealt out, showed no difference beyond
// noise.  Within 128 registers the bf16 form spills; at three workgroups per CU it does not.)
template <typename KT, int D>
__global__ __launch_bounds__(64 * kDecWaves, 3) void decode_kernel_alone(AttnArgs a)
{
    __shared__ DecMerge<kDecWaves, D> mg;
    decode_item<KT, 2, kDecWaves, D, false, false, true>(a, load_dec_item(a.dec + blockIdx.x / a.geo.Hkv), blockIdx.x % a.geo.Hkv, mg);
}

// Small decode-only batches are bound by their launches and by the chain of dependent reads at the start of an
// item.  Their fused form has one launch less and one link less: the items append the rows' new tokens themselves
// (decode_item<..., FUSED>: no append launch) and arrive as kernel arguments (no upload of the work lists and
// no read of a list from memory before the first page id can be asked for).
template <typename KT, int D>
__global__ __launch_bounds__(64 * kDecWaves) void decode_kernel_fused(AttnArgs a, SmallLists s)
{
    __shared__ DecMerge<kDecWaves, D> mg;
    const int w = blockIdx.x / a.geo.Hkv, g = blockIdx.x % a.geo.Hkv;
    const int first = s.wg[w], end = s.wg[w + 1];
    bool split = false;
    for (int i = first; i < end; ++i) {
        split |= s.dec[i].part >= 0;
        decode_item<KT, 2, kDecWaves, D, true, true, true>(a, s.dec[i], g, mg, i > first);
    }
    if (split && a.cmb_ctr) arrive_and_merge<D, 64 * kDecWaves, true>(a, s.dec + first, end - first, s.cmb, g);
}

// Merge of split rows as a launch (the rows from the device work list, or as kernel arguments behind the fused form): one
// workgroup per (row, head); its groups of D / 4 lanes take a chunk of eight
// splits each, the first group adds the chunks up in order.  (A row of 100 splits waits for two loads; one group
// walking all its splits took 10.6 us for three rows of 32 splits.)
__device__ __forceinline__ void combine_row(const AttnArgs& a, const CmbItem it)
{
    constexpr int kMaxGroups = 16;                         // 256 threads / (64 dims / 4)
    __shared__ f32x4 s_o[kMaxGroups][32];
    __shared__ float s_m[kMaxGroups], s_l[kMaxGroups];
    const int h = blockIdx.y, DQ = a.geo.D / 4, groups = 256 / DQ;
    const int grp = threadIdx.x / DQ, lane = threadIdx.x % DQ;
    const SplitParts parts(a, it.part_begin, it.n_split);
    SplitSum sum;
    for (int k0 = 0; k0 < it.n_split; k0 += groups * kMergeChunk) {
        const int mine = k0 + grp * kMergeChunk;
        if (mine < it.n_split) {
            const SplitSum c = sum_chunk(load_chunk(parts, mine, it.n_split, h, 4 * lane), mine, it.n_split);
            s_o[grp][lane] = c.o;
            if (lane == 0) { s_m[grp] = c.m; s_l[grp] = c.l; }
        }
        __syncthreads();
        if (grp == 0) {
            for (int j = 0; j < groups && k0 + j * kMergeChunk < it.n_split; ++j) {
                SplitSum c;
                c.m = s_m[j]; c.l = s_l[j]; c.o = s_o[j][lane];
                sum.add(c);
            }
        }
        __syncthreads();
    }
    if (grp == 0) store_merged(a, sum, it.row, h, 4 * lane);
}
__global__ __launch_bounds__(256) void combine_kernel(AttnArgs a) { combine_row(a, a.cmb[blockIdx.x]); }
struct SmallRows { CmbItem row[kSmallCmb]; };
__global__ __launch_bounds__(256) void combine_kernel_fused(AttnArgs a, SmallRows s) { combine_row(a, s.row[blockIdx.x]); }

template <typename KT, int D>
static int launch_decode_t(const AttnArgs& a, hipStream_t st, hipEvent_t done)
{
    dim3 grid((unsigned)(a.dec_wg ? a.n_dec_wg : a.n_dec) * (unsigned)a.geo.Hkv), block(64 * kDecWaves);
    switch (a.dec_nbuf) {
    case 3: return launch_kernel(decode_kernel<KT, 3, D>, grid, block, st, done, a);
    case 4: return launch_kernel(decode_kernel<KT, 4, D>, grid, block, st, done, a);
    default:
        if (a.dec_wg || a.cmb_ctr || (a.n_queue > 0 && a.geo.G > 8)) return launch_kernel(decode_kernel_lean_merging<KT, D>, grid, block, st, done, a);
        if constexpr (D == 128) {
            if (a.n_queue > 0) return launch_kernel(decode_kernel_lean<KT, D>, grid, block, st, done, a);   // (queues: the tiles of a co-resident launch)
        }
        return launch_kernel(decode_kernel_alone<KT, D>, grid, block, st, done, a);
    }
}

template <typename KT, int D>
static int resident_t(int nbuf)
{
    int per_cu = 0;
    hipError_t e;
    switch (nbuf) {
    case 3: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, decode_kernel<KT, 3, D>, 64 * kDecWaves, 0); break;
    case 4: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, decode_kernel<KT, 4, D>, 64 * kDecWaves, 0); break;
    default:
        if constexpr (D == 64) return decode_places_per_cu(D);     // (no resident prefill workgroups, so no decode_kernel_lean)
        else e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, decode_kernel_lean<KT, D>, 64 * kDecWaves, 0);
        break;
    }
    return e == hipSuccess ? per_cu : 0;
}

int decode_resident_workgroups(int kv_dtype, int nbuf, int head_dim)
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    int per_cu;
    if (head_dim == 64) per_cu = kv_dtype == TS_FP8_E4M3 ? resident_t<uint8_t, 64>(nbuf) : resident_t<uint16_t, 64>(nbuf);
    else per_cu = kv_dtype == TS_FP8_E4M3 ? resident_t<uint8_t, 128>(nbuf) : resident_t<uint16_t, 128>(nbuf);
    return cus * per_cu;
}

int launch_decode(const AttnArgs& a, void* stream, void* done)
{
    if (a.n_dec <= 0) return (int)hipSuccess;
    if ((a.geo.D != 128 && a.geo.D != 64) || a.geo.q_dtype != TS_BF16) return (int)hipErrorInvalidValue;
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t ev = (hipEvent_t)done;
    if (a.geo.kv_dtype == TS_BF16) return a.geo.D == 64 ? launch_decode_t<uint16_t, 64>(a, st, ev) : launch_decode_t<uint16_t, 128>(a, st, ev);
    if (a.geo.kv_dtype == TS_FP8_E4M3) return a.geo.D == 64 ? launch_decode_t<uint8_t, 64>(a, st, ev) : launch_decode_t<uint8_t, 128>(a, st, ev);
    return (int)hipErrorInvalidValue;
}

template <typename KT, int D>
static int launch_fused_t(const AttnArgs& a, const SmallLists& s, hipStream_t st, hipEvent_t done)
{
    dim3 grid((unsigned)s.n_wg * (unsigned)a.geo.Hkv), block(64 * kDecWaves);
    const bool merge = s.n_cmb > 0 && !a.cmb_ctr;
    const int e = launch_kernel(decode_kernel_fused<KT, D>, grid, block, st, merge ? nullptr : done, a, s);
    if (e != (int)hipSuccess || !merge) return e;
    SmallRows rows;
    std::copy(s.cmb, s.cmb + kSmallCmb, rows.row);
    return launch_kernel(combine_kernel_fused, dim3((unsigned)s.n_cmb, (unsigned)a.geo.Hq), dim3(256), st, done, a, rows);
}

int launch_decode_fused(const AttnArgs& a, const SmallLists& s, void* stream, void* done)
{
    if (s.n_dec <= 0) return (int)hipSuccess;
    if (s.n_dec > kSmallDec || s.n_cmb > kSmallCmb || !a.k_new || !a.v_new) return (int)hipErrorInvalidValue;
    if ((a.geo.D != 128 && a.geo.D != 64) || a.geo.q_dtype != TS_BF16) return (int)hipErrorInvalidValue;
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t ev = (hipEvent_t)done;
    if (a.geo.kv_dtype == TS_BF16) return a.geo.D == 64 ? launch_fused_t<uint16_t, 64>(a, s, st, ev) : launch_fused_t<uint16_t, 128>(a, s, st, ev);
    if (a.geo.kv_dtype == TS_FP8_E4M3) return a.geo.D == 64 ? launch_fused_t<uint8_t, 64>(a, s, st, ev) : launch_fused_t<uint8_t, 128>(a, s, st, ev);
    return (int)hipErrorInvalidValue;
}

int launch_combine(const AttnArgs& a, void* stream, void* done)
{
    if (a.n_cmb <= 0) return (int)hipSuccess;
    return launch_kernel(combine_kernel, dim3((unsigned)a.n_cmb, (unsigned)a.geo.Hq), dim3(256), (hipStream_t)stream, (hipEvent_t)done, a);
}

}  // namespace ts
