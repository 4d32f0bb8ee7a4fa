// Step a1: write the iteration's new K/V rows into the paged cache.
//
// Prefill builds cache entries for all input tokens, a decode iteration adds the entry of the
// last token (paper Sec. 2.1); in a Convertible Decoder both kinds of rows arrive in one batch
// (Sec. 3.4).  Kernels:
//   - append_small_kernel: batches of few sequences, see there;
//   - append_run_kernel: fp32 caches, see there;
//   - append_token_kernel: one workgroup per new token of a short sequence (decode rows): looks up the
//     token's page and slot and scatters its Hkv x D values of K (16-byte dim-chunks) and V
//     (token-fastest tile) into place.  The copy of the call's work lists from the pinned staging
//     buffer to device memory can ride along as extra workgroups of the same launch (a launch costs
//     more than either job: a decode step then has one kernel less in front of the scan);
//   - append_tile_kernel: one workgroup per (cache page, KV head) of a chunk: loads the page's up
//     to 16 new rows with full 256-byte reads, turns them into the K tile and -- through LDS --
//     into the token-fastest V tile, and writes whole 16-byte vectors.  (Scattering a chunk token
//     by token wrote 5.5x the new bytes: every 2-byte V element dirtied its own cache sector.)
// All convert to the cache element type with the same functions, so the bytes are identical.
#include "ts_device.h"
#include "ts_launch.h"

namespace ts {

// The work-list upload that rides along in the workgroups from first_block on.
__device__ __forceinline__ void upload_lists(const AppendArgs& a, int first_block)
{
    const int64_t stride = (int64_t)a.up_blocks * blockDim.x;
    for (int64_t i = (int64_t)((int)blockIdx.x - first_block) * blockDim.x + threadIdx.x; i < a.up_n16; i += stride)
        ((uint4*)a.up_dst)[i] = ((const uint4*)a.up_src)[i];
}

// bf16 source rows; DST: cache element type (uint16_t bf16 bits, uint8_t e4m3).
template <typename DST>
__global__ __launch_bounds__(256) void append_token_kernel(AppendArgs a)
{
    if ((int)blockIdx.x >= a.n_apr) { upload_lists(a, a.n_apr); return; }
    const AppRow r = a.apr[blockIdx.x];
    const int row = r.row, pos = r.pos;
    const int Hkv = a.geo.Hkv, D = a.geo.D;
    constexpr int X = 16 / (int)sizeof(DST);       // elements per 16-byte dim-chunk
    const int n_elems = Hkv * D;
    const uint16_t* ks = (const uint16_t*)a.k_new + (int64_t)row * n_elems;
    const uint16_t* vs = (const uint16_t*)a.v_new + (int64_t)row * n_elems;
    DST* kc = (DST*)a.k_cache;
    DST* vc = (DST*)a.v_cache;
    // (the values are requested before the page id is needed: the two loads wait together)
    const int32_t* page_ptr = a.block_table + (int64_t)r.seq * a.geo.max_pages + (pos >> 4);
    const int slot = pos & 15;
    for (int e0 = 0; e0 < n_elems; e0 += 4 * 256) {
        uint16_t kv[4], vv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = e0 + i * 256 + threadIdx.x;
            kv[i] = e < n_elems ? ks[e] : (uint16_t)0;
            vv[i] = e < n_elems ? vs[e] : (uint16_t)0;
        }
        const int64_t page = *page_ptr;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = e0 + i * 256 + threadIdx.x;
            if (e >= n_elems) continue;
            const int g = e / D, dim = e - g * D;
            const int64_t tile = tile_elem_base(page, Hkv, g, D);
            const int64_t kidx = tile + (dim / X) * (kPage * X) + slot * X + (dim % X);
            const int64_t vidx = tile + dim * kPage + slot;
            if constexpr (sizeof(DST) == 1) {
                const float kf = bf16_bits_to_float(kv[i]) / a.k_scale[g];
                const float vf = bf16_bits_to_float(vv[i]) / a.v_scale[g];
                __builtin_nontemporal_store((uint8_t)float_to_e4m3_bits(kf), &kc[kidx]);
                __builtin_nontemporal_store((uint8_t)float_to_e4m3_bits(vf), &vc[vidx]);
            } else {
                __builtin_nontemporal_store((DST)kv[i], &kc[kidx]);   // same element type: plain copy of the bits
                __builtin_nontemporal_store((DST)vv[i], &vc[vidx]);
            }
        }
    }
}

// fp32 cache, the new tokens of one page for one KV head: waves 0-1 write K (16-byte chunks, neighbouring slots
// together), waves 2-3 write V: a thread holds all slots of one dim and stores them as whole 16-byte pieces, so a
// page's V lines leave the L2 complete.  (One token per workgroup stored V in single 4-byte pieces, 64 bytes apart.)
template <int D>
__device__ __forceinline__ void append_page_f32(const AppendArgs& a, const AppTile it, int g)
{
    const int Hkv = a.geo.Hkv;
    const int64_t page = a.block_table[(int64_t)it.seq * a.geo.max_pages + it.page_idx];
    const int64_t tile = tile_elem_base(page, Hkv, g, D);
    const int lo = it.slots & 255, hi = it.slots >> 8;
    const int64_t src0 = ((int64_t)it.row_slot0 * Hkv + g) * D, row_step = (int64_t)Hkv * D;
    const int tid = threadIdx.x;
    if (tid < 128) {
        const float* src = (const float*)a.k_new;
        float* kt = (float*)a.k_cache + tile;
#pragma unroll
        for (int i = tid; i < 4 * D; i += 128) {       // (chunk of 4 dims, slot): slots fastest, as in the tile
            const int c = i >> 4, slot = i & 15;
            if (slot >= lo && slot < hi) *(f32x4*)(kt + i * 4) = *(const f32x4_u*)(src + src0 + slot * row_step + 4 * c);
        }
        return;
    }
    const int dim = tid - 128;
    if (dim >= D) return;
    const float* src = (const float*)a.v_new + src0 + dim;
    float* vt = (float*)a.v_cache + tile + dim * kPage;
    float v[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) v[s] = s >= lo && s < hi ? src[s * row_step] : 0.f;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if (4 * b >= lo && 4 * b + 4 <= hi) *(f32x4*)(vt + 4 * b) = f32x4{v[4 * b], v[4 * b + 1], v[4 * b + 2], v[4 * b + 3]};
        else
#pragma unroll
            for (int s = 4 * b; s < 4 * b + 4; ++s)
                if (s >= lo && s < hi) vt[s] = v[s];
    }
}

// Sixteen fp32 values -> sixteen e4m3 bytes (four words, value i in byte i % 4 of word i / 4), the same bytes as
// float_to_e4m3_bits gives.  The hardware conversion (two values per instruction, nearest-even, denormals and
// -0 as the definition wants) answers a value beyond the format's range, and any NaN, with the byte 0xFF; for
// every one of the 2^32 inputs it agrees with float_to_e4m3_bits once the value has been clamped to +-448,
// except on NaNs (compared exhaustively on the GPU).  So: clamp, convert, and take the integer encoder when
// any lane of the wave holds a NaN (rare; the branch is wave-uniform).
__device__ __forceinline__ void encode_e4m3x16(const float (&x)[16], uint32_t (&w)[4])
{
    bool nan = false;
#pragma unroll
    for (int i = 0; i < 16; ++i) nan |= x[i] != x[i];
    if (__any(nan)) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            w[j] = float_to_e4m3_bits(x[4 * j]) | (float_to_e4m3_bits(x[4 * j + 1]) << 8) |
                   (float_to_e4m3_bits(x[4 * j + 2]) << 16) | (float_to_e4m3_bits(x[4 * j + 3]) << 24);
        return;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float a = __builtin_amdgcn_fmed3f(x[4 * j], -448.0f, 448.0f), b = __builtin_amdgcn_fmed3f(x[4 * j + 1], -448.0f, 448.0f);
        const float c = __builtin_amdgcn_fmed3f(x[4 * j + 2], -448.0f, 448.0f), d = __builtin_amdgcn_fmed3f(x[4 * j + 3], -448.0f, 448.0f);
        int v = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
        v = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, v, true);
        w[j] = (uint32_t)v;
    }
}

// bf16 source rows, head dim D = 64 or 128; DST = uint16_t (bf16 cache) or uint8_t (e4m3 cache).
// One cache page for one KV head: thread (t = tid / (D/8), c = tid % (D/8)) loads the 16 bytes (dims 8c .. 8c+7) of slot t's K and V row
// (head dim 64: the first 128 threads).
template <typename DST, int D>
__device__ __forceinline__ void append_page(const AppendArgs& a, const AppTile it, int g)
{
    constexpr int CPR = D / 8;                         // 16-byte pieces per source row
    constexpr int kRowPad = D + 8;                     // LDS row stride in elements: avoids bank conflicts
    __shared__ __align__(16) uint16_t ks[16 * kRowPad];
    __shared__ __align__(16) uint16_t vs[16 * kRowPad];
    const int Hkv = a.geo.Hkv;
    const int slot_lo = it.slots & 255, slot_hi = it.slots >> 8;
    const int tid = threadIdx.x, t = tid / CPR, c = tid % CPR;
    const bool loader = tid < kPage * CPR;
    const int64_t page = a.block_table[(int64_t)it.seq * a.geo.max_pages + it.page_idx];
    const bool mine = loader && t >= slot_lo && t < slot_hi;
    uint4 kv = make_uint4(0, 0, 0, 0), vv = kv;
    if (mine) {
        const int64_t src = ((int64_t)(it.row_slot0 + t) * Hkv + g) * D + 8 * c;
        kv = *(const uint4*)((const uint16_t*)a.k_new + src);
        vv = *(const uint4*)((const uint16_t*)a.v_new + src);
    }
    if (loader) {
        *(uint4*)(vs + t * kRowPad + 8 * c) = vv;
        if constexpr (sizeof(DST) == 1) *(uint4*)(ks + t * kRowPad + 8 * c) = kv;
    }
    __syncthreads();
    const bool full = slot_lo == 0 && slot_hi == kPage;

    if constexpr (sizeof(DST) == 2) {
        uint16_t* kt = (uint16_t*)a.k_cache + tile_elem_base(page, Hkv, g, D);
        uint16_t* vt = (uint16_t*)a.v_cache + tile_elem_base(page, Hkv, g, D);
        // K tile [D/8 chunks][16 slots][8]: this thread's own 16 bytes
        if (mine) store_nt(kt + (c * 16 + t) * 8, kv);
        // V tile [D dims][16 slots]: thread (dim = tid / 2, half = tid % 2) gathers 8 slots of one dim
        const int dim = tid >> 1, hf = tid & 1;
        if (dim < D) {
            uint16_t e[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) e[i] = vs[(8 * hf + i) * kRowPad + dim];
            uint16_t* dst = vt + dim * kPage + 8 * hf;
            if (full) {
                store_nt(dst, make_uint4(e[0] | ((uint32_t)e[1] << 16), e[2] | ((uint32_t)e[3] << 16),
                                         e[4] | ((uint32_t)e[5] << 16), e[6] | ((uint32_t)e[7] << 16)));
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (8 * hf + i >= slot_lo && 8 * hf + i < slot_hi) __builtin_nontemporal_store(e[i], &dst[i]);
            }
        }
    } else {
        uint8_t* kt = (uint8_t*)a.k_cache + tile_elem_base(page, Hkv, g, D);
        uint8_t* vt = (uint8_t*)a.v_cache + tile_elem_base(page, Hkv, g, D);
        const float kscale = a.k_scale[g], vscale = a.v_scale[g];
        if (tid < D) {
            // K tile [D/16 chunks of 16 dims][16 slots][16]: thread (chunk = tid / 16, slot = tid % 16)
            const int c16 = tid >> 4, slot = tid & 15;
            if (slot >= slot_lo && slot < slot_hi) {
                float x[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) x[i] = bf16_bits_to_float(ks[slot * kRowPad + 16 * c16 + i]) / kscale;
                uint32_t w[4];
                encode_e4m3x16(x, w);
                store_nt(kt + (c16 * 16 + slot) * 16, make_uint4(w[0], w[1], w[2], w[3]));
            }
        } else if (tid < 2 * D) {
            // V tile [D dims][16 slots]: thread dim = tid - D gathers the 16 slots of one dim
            const int dim = tid - D;
            float x[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = bf16_bits_to_float(vs[i * kRowPad + dim]) / vscale;
            uint32_t w[4];
            encode_e4m3x16(x, w);
            uint8_t* dst = vt + dim * kPage;
            if (full) {
                store_nt(dst, make_uint4(w[0], w[1], w[2], w[3]));
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (i >= slot_lo && i < slot_hi)
                        __builtin_nontemporal_store((uint8_t)(w[i >> 2] >> (8 * (i & 3))), &dst[i]);
            }
        }
    }
}

template <typename DST, int D>
__device__ __forceinline__ void append_any_page(const AppendArgs& a, const AppTile it, int g)
{
    if constexpr (sizeof(DST) == 4) append_page_f32<D>(a, it, g);
    else append_page<DST, D>(a, it, g);
}

// Page-wise list of the plan.
template <typename DST, int D>
__global__ __launch_bounds__(256) void append_tile_kernel(AppendArgs a)
{
    const int pages = a.n_apt * a.geo.Hkv;
    if ((int)blockIdx.x >= pages) upload_lists(a, pages);
    else append_page<DST, D>(a, a.apt[blockIdx.x / a.geo.Hkv], blockIdx.x % a.geo.Hkv);
}

// fp32 cache: one record per run of new tokens of a page.
template <int D>
__global__ __launch_bounds__(256) void append_run_kernel(AppendArgs a)
{
    const int n = a.n_apr * a.geo.Hkv;
    if ((int)blockIdx.x >= n) { upload_lists(a, n); return; }
    const AppRow r = a.apr[blockIdx.x / a.geo.Hkv];
    const int lo = r.pos & (kPage - 1);
    append_page_f32<D>(a, AppTile{r.seq, r.pos >> 4, lo | (lo + r.run) << 8, r.row - lo}, blockIdx.x % a.geo.Hkv);
}

// Batches of few sequences: every new token goes page by page (a decode row is a page with one new token), and the
// sequences' descriptions arrive as kernel arguments: one launch instead of two for a batch of both kinds, and no
// list to read over PCIe before the first page id can be asked for.  A workgroup finds its sequence by comparing its
// page number with the sequences' first page numbers, one per lane (a sequence without new tokens has none and shares
// the number of the next one: the last match counts).
template <typename DST, int D>
__global__ __launch_bounds__(256) void append_small_kernel(AppendArgs a, AppendSeqs s)
{
    const int Hkv = a.geo.Hkv;
    const int u = blockIdx.x / Hkv, g = blockIdx.x % Hkv;
    if (u >= s.n_pages) { upload_lists(a, s.n_pages * Hkv); return; }
    const int lane = threadIdx.x & 63;
    int i = -1;
#pragma unroll
    for (int b = 0; b < kAppendSeqs; b += 64)
        i += __builtin_popcountll(__ballot(b + lane < s.n && s.seq[min(b + lane, kAppendSeqs - 1)].first_page <= u));
    const AppendSeq q = s.seq[i];
    const int q_len = s.seq[i + 1].row0 - q.row0, page_idx = (q.prefix >> 4) + u - q.first_page;
    const int lo = max(q.prefix - page_idx * kPage, 0), hi = min(q.prefix + q_len - page_idx * kPage, kPage);
    append_any_page<DST, D>(a, AppTile{i, page_idx, lo | hi << 8, q.row0 + page_idx * kPage - q.prefix}, g);
}

template <typename DST, int D>
static int launch_append_small(const AppendArgs& a, const AppendSeqs& s, hipStream_t st, hipEvent_t done)
{
    const dim3 grid((unsigned)s.n_pages * (unsigned)a.geo.Hkv + (unsigned)a.up_blocks);
    return launch_kernel(append_small_kernel<DST, D>, grid, dim3(256), st, done, a, s);
}

int launch_append_few(const AppendArgs& a, const AppendSeqs& s, void* stream, void* done)
{
    if (s.n <= 0) return (int)hipSuccess;
    if (s.n > kAppendSeqs || s.n_pages <= 0 || (a.geo.D != 128 && a.geo.D != 64)) return (int)hipErrorInvalidValue;
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t ev = (hipEvent_t)done;
    const bool d128 = a.geo.D == 128;
    if (a.geo.q_dtype == TS_F32 && a.geo.kv_dtype == TS_F32)
        return d128 ? launch_append_small<float, 128>(a, s, st, ev) : launch_append_small<float, 64>(a, s, st, ev);
    if (a.geo.q_dtype == TS_BF16 && a.geo.kv_dtype == TS_BF16)
        return d128 ? launch_append_small<uint16_t, 128>(a, s, st, ev) : launch_append_small<uint16_t, 64>(a, s, st, ev);
    if (a.geo.q_dtype == TS_BF16 && a.geo.kv_dtype == TS_FP8_E4M3)
        return d128 ? launch_append_small<uint8_t, 128>(a, s, st, ev) : launch_append_small<uint8_t, 64>(a, s, st, ev);
    return (int)hipErrorInvalidValue;
}

int launch_append(const AppendArgs& args, void* stream, void* done)
{
    if (args.total_tokens <= 0) return (int)hipSuccess;
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t ev = args.n_apt > 0 ? nullptr : (hipEvent_t)done;     // (of the token-wise launch)
    dim3 block(256);
    AppendArgs a = args;
    int e = (int)hipSuccess;
    // the upload (if any) rides in the first launch, which then reads its own list from the staging buffer
    if (a.up_blocks > 0) {
        if (a.n_apr > 0) a.apr = a.apr_host; else a.apt = a.apt_host;
    }
    if (a.n_apr > 0 && a.geo.q_dtype == TS_F32) {
        if (a.geo.kv_dtype != TS_F32 || (a.geo.D != 128 && a.geo.D != 64)) return (int)hipErrorInvalidValue;
        const int64_t most = kMaxWorkgroups > a.geo.Hkv ? kMaxWorkgroups / a.geo.Hkv : 1;
        for (int64_t first = 0, left = a.n_apr; left > 0 && e == (int)hipSuccess; first += most, left -= most) {
            AppendArgs part = a;
            part.apr = a.apr + first;
            part.n_apr = (int32_t)(left < most ? left : most);
            if (first > 0) part.up_blocks = 0;
            const dim3 grid((unsigned)part.n_apr * (unsigned)a.geo.Hkv + (unsigned)part.up_blocks);
            const hipEvent_t pe = left <= most ? ev : nullptr;
            if (a.geo.D == 128) e = launch_kernel(append_run_kernel<128>, grid, block, st, pe, part);
            else e = launch_kernel(append_run_kernel<64>, grid, block, st, pe, part);
        }
    } else if (a.n_apr > 0) {
        dim3 grid((unsigned)(a.n_apr + a.up_blocks));
        if (a.geo.q_dtype == TS_BF16 && a.geo.kv_dtype == TS_BF16)
            e = launch_kernel(append_token_kernel<uint16_t>, grid, block, st, ev, a);
        else if (a.geo.q_dtype == TS_BF16 && a.geo.kv_dtype == TS_FP8_E4M3)
            e = launch_kernel(append_token_kernel<uint8_t>, grid, block, st, ev, a);
        else
            return (int)hipErrorInvalidValue;
    }
    if (a.n_apr > 0) {
        a.up_blocks = 0;                               // done; the page-wise kernel finds its list on the device
        a.apt = args.apt;
    }
    if (e != (int)hipSuccess || a.n_apt == 0) return e;
    if (a.geo.q_dtype != TS_BF16 || (a.geo.D != 128 && a.geo.D != 64)) return (int)hipErrorInvalidValue;
    if (a.geo.kv_dtype != TS_BF16 && a.geo.kv_dtype != TS_FP8_E4M3) return (int)hipErrorInvalidValue;
    dim3 tgrid((unsigned)a.n_apt * (unsigned)a.geo.Hkv + (unsigned)a.up_blocks);
    const bool bf = a.geo.kv_dtype == TS_BF16;
    const hipEvent_t te = (hipEvent_t)done;
    if (a.geo.D == 128) {
        if (bf) return launch_kernel(append_tile_kernel<uint16_t, 128>, tgrid, block, st, te, a);
        return launch_kernel(append_tile_kernel<uint8_t, 128>, tgrid, block, st, te, a);
    }
    if (bf) return launch_kernel(append_tile_kernel<uint16_t, 64>, tgrid, block, st, te, a);
    return launch_kernel(append_tile_kernel<uint8_t, 64>, tgrid, block, st, te, a);
}

}  // namespace ts
