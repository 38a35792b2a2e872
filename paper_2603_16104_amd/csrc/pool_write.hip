// Scatter of new tokens' K/V into the pool's block format (one workgroup per touched page and KV
// head).  bf16 pools: plain re-ordering.  fp8 pools: per-block amax, scale = amax/448, codes =
// round-to-nearest-even(x / scale) saturated to +-448 (OCP e4m3), all in float.  A block that is
// continued (the call starts at first_slot > 0 of its first page) keeps a running scale:
// scale' = max(scale, amax_new/448); when the scale grows, the codes already in the slots below
// first_slot are re-encoded as RNE(value(code) * scale / scale'); the scale never shrinks.
// (The "compute a prefix's KV once and keep it in GPU memory" step of Section 5, "Proactive Cache
// Management", seen from the pool.)
// Also here, all small: the one-token-per-sequence form of the writer for decode steps, whole-page
// copies (copy-on-write), the fp8 -> bf16 pre-pass of prefill over fp8 pools, the copy kernel that
// replaces small host-to-device DMA copies, and the in-place update of a growing decode plan.
#include <algorithm>
#include <type_traits>

#include "hkv_device.h"

namespace hkv {

namespace {

__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp<kQuadXor1>(v));
    v = fmaxf(v, dpp<kQuadXor2>(v));
    v = fmaxf(v, dpp<kRor4>(v));
    v = fmaxf(v, dpp<kRor8>(v));
    return rows_max(v);
}

__device__ __forceinline__ uint32_t quant4(float a, float b, float c, float d, float scale) {
    auto q = [scale](float x) { return fminf(fmaxf(x / scale, -448.0f), 448.0f); };
    int p = 0;
    p = __builtin_amdgcn_cvt_pk_fp8_f32(q(a), q(b), p, false);
    p = __builtin_amdgcn_cvt_pk_fp8_f32(q(c), q(d), p, true);
    return (uint32_t)p;
}

// The same codes for bf16 values x and a scale of amax / 448 of such values, |x| <= amax, from the scale's reciprocal
// (correctly rounded): product, remainder, correction.  For every such pair with a scale in [2^-60, 2^60] (5.3e8 pairs, all
// of them tried) the quotient equals the division's bit for bit wherever it is at least 2^-11 in magnitude; below 2^-10
// both round to zero with the sign of x.  Four instructions instead of about ten, two of them slow ones.
__device__ __forceinline__ uint32_t quant4_by(float a, float b, float c, float d, float scale, float inv) {
    auto q = [scale, inv](float x) {
        const float y = x * inv;
        const float z = __builtin_copysignf(__builtin_fmaf(__builtin_fmaf(-y, scale, x), inv, y), x);
        return fminf(fmaxf(z, -448.0f), 448.0f);
    };
    int p = 0;
    p = __builtin_amdgcn_cvt_pk_fp8_f32(q(a), q(b), p, false);
    p = __builtin_amdgcn_cvt_pk_fp8_f32(q(c), q(d), p, true);
    return (uint32_t)p;
}

// One workgroup's work.  single: one token per block (source row pi goes to slot one_slot of block
// `page`) instead of a run of tokens over consecutive blocks.
template <int DT>
__device__ __forceinline__ void pool_write_block(const PoolWriteLaunch &a, const int pi, const int page, const int h, const bool single,
                                                 const int one_slot) {
    __shared__ uint16_t sV[kPage][kHeadDim + 8];
    __shared__ float sRed[2][4];
    __shared__ float sScale[2], sOld[2], sInv[2];

    const int tid = threadIdx.x;
    const int slot = tid >> 4, d0 = (tid & 15) * 8;
    const int tok = single ? pi : pi * kPage + slot - a.first_slot;  // source row of this thread's slot
    const bool valid = single ? slot == one_slot : (tok >= 0 && tok < a.n_tokens);
    const size_t blk = ((size_t)page * a.num_kv_heads + h) * kBlockElems;

    u32x4 kw = {0u, 0u, 0u, 0u}, vw = {0u, 0u, 0u, 0u};
    if (valid) {
        const size_t src = (((size_t)tok * a.num_kv_heads + h) * kHeadDim + d0) * 2;
        kw = ld16(static_cast<const char *>(a.k_src) + src);
        vw = ld16(static_cast<const char *>(a.v_src) + src);
    }
    *reinterpret_cast<u32x4 *>(&sV[slot][d0]) = vw;

    // which slots of this page does the call write?  (contiguous range)
    const int s_lo = single ? one_slot : max(0, a.first_slot - pi * kPage);
    const int s_hi = single ? one_slot + 1 : min(kPage, a.first_slot + a.n_tokens - pi * kPage);  // exclusive

    if (DT == 0) {
        if (valid) {
            uint16_t *kdst = static_cast<uint16_t *>(a.k_pages) + blk + (d0 >> 5) * (kPage * 32) + slot * 32 + (d0 & 31);
            *reinterpret_cast<u32x4 *>(kdst) = kw;
        }
        __syncthreads();
        const int d = tid >> 1, half = tid & 1;
        uint16_t *vdst = static_cast<uint16_t *>(a.v_pages) + blk + d * kPage + half * 8;
        if (s_lo <= half * 8 && s_hi >= half * 8 + 8) {
            u32x4 w;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                w[j] = (uint32_t)sV[half * 8 + 2 * j][d] | ((uint32_t)sV[half * 8 + 2 * j + 1][d] << 16);
            *reinterpret_cast<u32x4 *>(vdst) = w;
        } else {
            for (int j = 0; j < 8; ++j) {
                const int sl = half * 8 + j;
                if (sl >= s_lo && sl < s_hi) vdst[j] = sV[sl][d];
            }
        }
    } else {
        float kf[8], vf[8];
        float ka = 0.f, va = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            kf[2 * j] = __uint_as_float(kw[j] << 16);
            kf[2 * j + 1] = __uint_as_float(kw[j] & 0xFFFF0000u);
            vf[2 * j] = __uint_as_float(vw[j] << 16);
            vf[2 * j + 1] = __uint_as_float(vw[j] & 0xFFFF0000u);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            ka = fmaxf(ka, fabsf(kf[j]));
            va = fmaxf(va, fabsf(vf[j]));
        }
        ka = wave_max(ka);
        va = wave_max(va);
        if ((tid & 63) == 0) {
            sRed[0][tid >> 6] = ka;
            sRed[1][tid >> 6] = va;
        }
        __syncthreads();
        const bool append = s_lo > 0;  // slots below s_lo of this block hold codes of an earlier call
        if (tid < 2) {
            const float am = fmaxf(fmaxf(sRed[tid][0], sRed[tid][1]), fmaxf(sRed[tid][2], sRed[tid][3]));
            float *scales = tid ? a.v_scale : a.k_scale;
            float sc, old = 0.f;
            if (!append) {
                sc = am > 0.f ? am / 448.0f : 1.0f;
            } else {
                old = scales[(size_t)page * a.num_kv_heads + h];
                const float cand = am > 0.f ? am / 448.0f : 0.f;
                sc = old >= cand ? old : cand;  // an unset (NaN) old scale gives cand
                if (!(sc > 0.f)) sc = 1.0f;
            }
            sScale[tid] = sc;
            sOld[tid] = old;
            sInv[tid] = !append && sc >= 0x1p-60f && sc <= 0x1p60f ? 1.0f / sc : 0.f;  // 0: divide
            scales[(size_t)page * a.num_kv_heads + h] = sc;
        }
        __syncthreads();
        const float ksc = sScale[0], vsc = sScale[1], kinv = sInv[0], vinv = sInv[1];
        auto encode = [](const float (&x)[8], float sc, float inv) {
            u32x2 c;
            if (inv != 0.f) {  // the same for the whole workgroup
                c[0] = quant4_by(x[0], x[1], x[2], x[3], sc, inv);
                c[1] = quant4_by(x[4], x[5], x[6], x[7], sc, inv);
            } else {
                c[0] = quant4(x[0], x[1], x[2], x[3], sc);
                c[1] = quant4(x[4], x[5], x[6], x[7], sc);
            }
            return c;
        };
        const bool k_grew = append && ksc > sOld[0], v_grew = append && vsc > sOld[1];
        auto reencode4 = [](uint32_t w, float old, float sc) {  // four codes: value * old / sc, rounded again
            const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, false), hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, true);
            return quant4(lo[0] * old, lo[1] * old, hi[0] * old, hi[1] * old, sc);
        };
        if (k_grew && slot < s_lo) {
            uint8_t *kdst = static_cast<uint8_t *>(a.k_pages) + blk + (d0 >> 6) * (kPage * 64) + slot * 64 + (d0 & 63);
            u32x2 c = *reinterpret_cast<u32x2 *>(kdst);
            c[0] = reencode4(c[0], sOld[0], ksc);
            c[1] = reencode4(c[1], sOld[0], ksc);
            *reinterpret_cast<u32x2 *>(kdst) = c;
        }
        if (valid) {
            const u32x2 c = encode(kf, ksc, kinv);
            uint8_t *kdst = static_cast<uint8_t *>(a.k_pages) + blk + (d0 >> 6) * (kPage * 64) + slot * 64 + (d0 & 63);
            *reinterpret_cast<u32x2 *>(kdst) = c;
        }
        const int d = tid >> 1, half = tid & 1;
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = bf16_bits_to_float(sV[half * 8 + j][d]);
        const u32x2 c = encode(x, vsc, vinv);
        uint8_t *vdst = static_cast<uint8_t *>(a.v_pages) + blk + d * kPage + half * 8;
        if (s_lo <= half * 8 && s_hi >= half * 8 + 8) {
            *reinterpret_cast<u32x2 *>(vdst) = c;
        } else {
            u32x2 r = {0u, 0u};  // the earlier codes of these eight slots, re-encoded if the scale grew
            if (v_grew && half * 8 < s_lo) {
                r = *reinterpret_cast<u32x2 *>(vdst);
                r[0] = reencode4(r[0], sOld[1], vsc);
                r[1] = reencode4(r[1], sOld[1], vsc);
            }
            for (int j = 0; j < 8; ++j) {
                const int sl = half * 8 + j;
                if (sl >= s_lo && sl < s_hi)
                    vdst[j] = (uint8_t)(c[j >> 2] >> (8 * (j & 3)));
                else if (v_grew && sl < s_lo)
                    vdst[j] = (uint8_t)(r[j >> 2] >> (8 * (j & 3)));
            }
        }
    }
}

// K (v = false) or V of one block of an fp8 pool that the call writes whole, by one wavefront, without LDS or barriers: lane
// (row q of 16, column c) holds tokens 4 q .. 4 q + 3 of dims 8 c .. 8 c + 7, so that V's four codes of a dim make a word
// of one lane and its dimension-major order is a transposition of words between the four rows, in the vector ALU.  Bound by the
// chain load, maximum, quotients, store of one wavefront (up to about 4000 tokens x 8 heads a launch has all of them on the chip at
// once): 4096 tokens 5.9 -> 5.1 us, 8192 tokens 11.0 -> 9.1 us against the general form, which passes V through LDS and the
// maxima over two barriers.  (bf16 pools have neither maxima nor codes: the same form took 5.9 instead of 5.4 us there.)
__device__ __forceinline__ void transpose_rows(uint32_t (&x)[4]) {  // word d of row q <-> word q of row d
    const auto a = __builtin_amdgcn_permlane32_swap(x[0], x[2], false, false), b = __builtin_amdgcn_permlane32_swap(x[1], x[3], false, false);
    const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false), d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    x[0] = c[0];
    x[1] = c[1];
    x[2] = d[0];
    x[3] = d[1];
}
__device__ __forceinline__ void write_whole_fp8_block(const PoolWriteLaunch &a, const int pi, const int page, const int h, const bool v) {
    const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
    const size_t blk = ((size_t)page * a.num_kv_heads + h) * kBlockElems;
    const char *src = static_cast<const char *>(v ? a.v_src : a.k_src) +
                      (((size_t)(pi * kPage + 4 * q - a.first_slot) * a.num_kv_heads + h) * kHeadDim + 8 * c) * 2;
    u32x4 w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = ld16(src + (size_t)i * a.num_kv_heads * kHeadDim * 2);
    float x[4][8];
    float am = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            x[i][2 * j] = __uint_as_float(w[i][j] << 16);
            x[i][2 * j + 1] = __uint_as_float(w[i][j] & 0xFFFF0000u);
            am = fmaxf(am, fabsf(x[i][2 * j]));
            am = fmaxf(am, fabsf(x[i][2 * j + 1]));
        }
    am = wave_max(am);
    const float sc = am > 0.f ? am / 448.0f : 1.0f;
    const float inv = sc >= 0x1p-60f && sc <= 0x1p60f ? 1.0f / sc : 0.f;  // 0: divide
    if (lane == 0) (v ? a.v_scale : a.k_scale)[(size_t)page * a.num_kv_heads + h] = sc;
    auto encode = [&](float x0, float x1, float x2, float x3) {
        return inv != 0.f ? quant4_by(x0, x1, x2, x3, sc, inv) : quant4(x0, x1, x2, x3, sc);  // the same for the whole wavefront
    };
    if (!v) {
        uint8_t *dst = static_cast<uint8_t *>(a.k_pages) + blk + (c >> 3) * (kPage * 64) + 4 * q * 64 + (c & 7) * 8;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<u32x2 *>(dst + 64 * i) = u32x2{encode(x[i][0], x[i][1], x[i][2], x[i][3]), encode(x[i][4], x[i][5], x[i][6], x[i][7])};
        return;
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        uint32_t t[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) t[j] = encode(x[0][4 * e + j], x[1][4 * e + j], x[2][4 * e + j], x[3][4 * e + j]);
        transpose_rows(t);
        *reinterpret_cast<u32x4 *>(static_cast<uint8_t *>(a.v_pages) + blk + (8 * c + 4 * e + q) * kPage) = u32x4{t[0], t[1], t[2], t[3]};
    }
}

// A run of tokens: workgroup (block, head), or (PAIRS, large writes into fp8 pools) workgroup (block, pair of heads), of which
// wavefront w takes K (w even) or V (w odd) of head w / 2 of the pair; a block that the call writes in part, its first or its last one, goes the general way,
// the pair's second head by the workgroup in row n_pages + (whether it is the second such block) of the grid.
__device__ __forceinline__ bool writes_whole(const PoolWriteLaunch &a, const int pi) {
    return pi * kPage >= a.first_slot && a.first_slot + a.n_tokens >= (pi + 1) * kPage;
}
template <int DT, bool PAIRS>
__device__ __forceinline__ void pool_write_run(const PoolWriteLaunch &a, const int32_t *ids) {
    static_assert(DT == 1 || !PAIRS, "only fp8 blocks have the other form");
    if constexpr (!PAIRS) {
        pool_write_block<DT>(a, blockIdx.x, ids[blockIdx.x], blockIdx.y, false, 0);
        return;
    }
    const int x = blockIdx.x;
    const bool extra = x >= a.n_pages;
    const int pi = !extra ? x : (x == a.n_pages && !writes_whole(a, 0)) ? 0 : a.n_pages - 1;
    const int page = ids[pi], h0 = 2 * blockIdx.y;
    if (!extra && writes_whole(a, pi)) {
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), h = h0 + (wave >> 1);
        if (h < a.num_kv_heads) write_whole_fp8_block(a, pi, page, h, wave & 1);
    } else if (h0 + extra < a.num_kv_heads) {
        pool_write_block<1>(a, pi, page, h0 + extra, false, 0);
    }
}

template <int DT, bool PAIRS>
__global__ __launch_bounds__(256) void pool_write_kernel(PoolWriteLaunch a) {
    if (!PAIRS && a.slots)
        pool_write_block<DT>(a, blockIdx.x, a.page_ids[blockIdx.x], blockIdx.y, true, a.slots[blockIdx.x]);
    else
        pool_write_run<DT, PAIRS>(a, a.page_ids);
}

// A write of up to kMaxInlineWrite blocks (15 360 tokens): the block ids travel in the kernel arguments.  Through the
// staging ring a call was an upload kernel, this kernel and an event: 13 us per call back to back for 2 200 tokens x 8
// heads into an fp8 pool, 6.7 us this way (the launch itself is most of either).  The line is the 4 KiB of kernel
// arguments; larger calls go through the ring, where the two extra launches no longer matter.
template <int N>
struct PoolWriteInline {
    PoolWriteLaunch base;
    int32_t block[N];
};
static_assert(sizeof(PoolWriteInline<kMaxInlineWrite>) <= 4096, "kernel argument segment");
template <int DT, bool PAIRS, int N>
__global__ __launch_bounds__(256) void pool_write_inline_kernel(PoolWriteInline<N> a) {
    pool_write_run<DT, PAIRS>(a.base, a.block);
}

// The decode step's append for up to kMaxInlineAppend sequences: block ids and slots travel in the kernel
// arguments, so the call needs no staging buffer, no copy and no event.
template <int DT>
__global__ __launch_bounds__(256) void pool_append_inline_kernel(PoolAppendInline a) {
    const int pi = blockIdx.x;
    pool_write_block<DT>(a.base, pi, a.block[pi], blockIdx.y, true, a.slot[pi]);
}

// One workgroup per (pair, K or V): copies the page's blocks of all KV heads, 16 bytes per thread and
// step, and (fp8 pools) the page's scales.  Source and destination pages are distinct.
__global__ __launch_bounds__(256) void pool_copy_kernel(PoolCopyLaunch a) {
    const int pair = blockIdx.x, which = blockIdx.y;
    const int elem = a.pool.dtype == 0 ? 2 : a.pool.dtype == 1 ? 1 : 4;
    const size_t page_bytes = (size_t)a.blocks_per_page * a.pool.num_kv_heads * kBlockElems * elem;
    const char *base = static_cast<const char *>(which ? a.pool.v_pages : a.pool.k_pages);
    const uint4 *src = reinterpret_cast<const uint4 *>(base + (size_t)a.src[pair] * page_bytes);
    uint4 *dst = reinterpret_cast<uint4 *>(const_cast<char *>(base) + (size_t)a.dst[pair] * page_bytes);
    for (size_t i = threadIdx.x; i < page_bytes / 16; i += 256) dst[i] = src[i];
    if (a.pool.dtype == 1) {
        float *sc = const_cast<float *>(which ? a.pool.v_scale : a.pool.k_scale);
        const int per_page = a.blocks_per_page * a.pool.num_kv_heads;  // one scale per 16-token block and head
        for (int h = threadIdx.x; h < per_page; h += 256)
            sc[(size_t)a.dst[pair] * per_page + h] = sc[(size_t)a.src[pair] * per_page + h];
    }
}

// One workgroup per (scratch page, KV head): value = code * scale, rounded to bf16 (RNE), written in the
// bf16 block format.  A thread converts 8 consecutive codes of K and of V: in both formats they are 8
// consecutive elements (K: 8 dimensions of one slot inside a 64-byte chunk; V: 8 slots of one dimension).
__global__ __launch_bounds__(256) void pool_dequant_kernel(PoolDequantLaunch a) {
    const int i = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
    const int page = a.src_pages[i];
    const size_t src_blk = ((size_t)page * a.pool.num_kv_heads + h) * kBlockElems;
    const size_t dst_blk = ((size_t)i * a.pool.num_kv_heads + h) * kBlockElems;
    const float ks = a.pool.k_scale[(size_t)page * a.pool.num_kv_heads + h];
    const float vs = a.pool.v_scale[(size_t)page * a.pool.num_kv_heads + h];
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    auto convert = [](u32x2 w, float sc) {
        u32x4 o;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[j], false), hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[j], true);
            o[2 * j] = pack_bf16(lo[0] * sc, lo[1] * sc);
            o[2 * j + 1] = pack_bf16(hi[0] * sc, hi[1] * sc);
        }
        return o;
    };
    {   // K: fp8 element (slot t, dim d) at (d / 64) * 1024 + t * 64 + d % 64, bf16 at (d / 32) * 512 + t * 32 + d % 32
        const int e = 8 * tid, c = e >> 10, t = (e >> 6) & 15, d = 64 * c + (e & 63);
        const u32x2 w = *reinterpret_cast<const u32x2 *>(static_cast<const uint8_t *>(a.pool.k_pages) + src_blk + e);
        *reinterpret_cast<u32x4 *>(static_cast<uint16_t *>(a.k_dst) + dst_blk + (d >> 5) * 512 + t * 32 + (d & 31)) = convert(w, ks);
    }
    {   // V: element (slot t, dim d) at d * 16 + t in both formats
        const int e = 8 * tid;
        const u32x2 w = *reinterpret_cast<const u32x2 *>(static_cast<const uint8_t *>(a.pool.v_pages) + src_blk + e);
        *reinterpret_cast<u32x4 *>(static_cast<uint16_t *>(a.v_dst) + dst_blk + e) = convert(w, vs);
    }
}

// Plain copy of n16 16-byte pieces; the source may be pinned host memory (read over the host link).
__global__ __launch_bounds__(256) void upload_kernel(const uint4 *__restrict__ src, uint4 *__restrict__ dst, size_t n16) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}

__global__ __launch_bounds__(256) void plan_grow_inline_kernel(PlanGrowInline a) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t < a.n_grow) a.items[a.grow_items[t]].n_tokens += 1;
    if (t < a.n_req && a.new_block[t] >= 0) a.pages[a.block_pos[t]] = a.new_block[t];
}

// A decode step's append in one launch: workgroup (r, head) stores request r's new token and lengthens the
// item of that head in the request's leaf (grow_items is [request][head]); head 0 enters a new block id.
template <int DT>
__global__ __launch_bounds__(256) void decode_step_append_kernel(PoolAppendInline w, PlanGrowInline g) {
    const int r = blockIdx.x, h = blockIdx.y;
    pool_write_block<DT>(w.base, r, w.block[r], h, true, w.slot[r]);
    if (threadIdx.x == 0) g.items[g.grow_items[r * w.base.num_kv_heads + h]].n_tokens += 1;
    if (threadIdx.x == 1 && h == 0 && g.new_block[r] >= 0) g.pages[g.block_pos[r]] = g.new_block[r];
}

}  // namespace

hipError_t launch_decode_step_append(const PoolAppendInline &w, const PlanGrowInline &g, hipStream_t s) {
    if (w.base.n_pages <= 0) return hipSuccess;
    dim3 grid(w.base.n_pages, w.base.num_kv_heads), block(256);
    if (w.base.dtype == 0)
        hipLaunchKernelGGL(decode_step_append_kernel<0>, grid, block, 0, s, w, g);
    else
        hipLaunchKernelGGL(decode_step_append_kernel<1>, grid, block, 0, s, w, g);
    return hipGetLastError();
}

hipError_t launch_plan_grow_inline(const PlanGrowInline &a, hipStream_t s) {
    const int n = a.n_grow > a.n_req ? a.n_grow : a.n_req;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(plan_grow_inline_kernel, dim3((n + 255) / 256), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_pool_dequant(const PoolDequantLaunch &a, hipStream_t s) {
    if (a.n_pages <= 0) return hipSuccess;
    hipLaunchKernelGGL(pool_dequant_kernel, dim3(a.n_pages, a.pool.num_kv_heads), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_upload(const void *src, void *dst, size_t bytes, hipStream_t s) {
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    const unsigned blocks = (unsigned)std::min<size_t>((n16 + 255) / 256, 256);
    hipLaunchKernelGGL(upload_kernel, dim3(blocks), dim3(256), 0, s, static_cast<const uint4 *>(src),
                       static_cast<uint4 *>(dst), n16);
    return hipGetLastError();
}

hipError_t launch_pool_copy(const PoolCopyLaunch &a, hipStream_t s) {
    if (a.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(pool_copy_kernel, dim3(a.n, 2), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_pool_append_inline(const PoolAppendInline &a, hipStream_t s) {
    if (a.base.n_pages <= 0) return hipSuccess;
    dim3 grid(a.base.n_pages, a.base.num_kv_heads), block(256);
    if (a.base.dtype == 0)
        hipLaunchKernelGGL(pool_append_inline_kernel<0>, grid, block, 0, s, a);
    else
        hipLaunchKernelGGL(pool_append_inline_kernel<1>, grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_pool_write(const PoolWriteLaunch &a, hipStream_t s) {
    if (a.n_pages <= 0) return hipSuccess;
    // A wavefront per K or V of a block takes longer alone than the four of a workgroup together; from 400 blocks x heads on that no
    // longer counts (fp8, device time of a write, workgroup per block and head / this: 8 heads, 320 tokens 2.80 / 2.99 us, 500 3.10 /
    // 3.33, 1000 3.51 / 3.26, 4096 5.89 / 5.08; 2 heads, 2000 tokens 2.88 / 3.06, 4096 3.20 / 3.22, 8192 3.99 / 3.72; 1 head, half
    // of whose wavefronts would idle, 8192 3.19 / 3.36).
    const bool pairs = a.dtype == 1 && !a.slots && a.num_kv_heads > 1 && (int64_t)a.n_pages * a.num_kv_heads >= 400;
    const int in_part = a.n_pages == 1 ? (a.first_slot > 0 || a.n_tokens < kPage) : (a.first_slot > 0) + ((a.first_slot + a.n_tokens) % kPage != 0);
    const dim3 grid(a.n_pages + (pairs ? in_part : 0), pairs ? (a.num_kv_heads + 1) / 2 : a.num_kv_heads), block(256);
    if (a.host_ids) {
        auto go = [&](auto room) {
            constexpr int N = decltype(room)::value;
            PoolWriteInline<N> w;
            w.base = a;
            w.base.host_ids = nullptr;
            std::copy(a.host_ids, a.host_ids + a.n_pages, w.block);
            std::fill(w.block + a.n_pages, w.block + N, 0);
            if (a.dtype == 0)
                hipLaunchKernelGGL((pool_write_inline_kernel<0, false, N>), grid, block, 0, s, w);
            else if (!pairs)
                hipLaunchKernelGGL((pool_write_inline_kernel<1, false, N>), grid, block, 0, s, w);
            else
                hipLaunchKernelGGL((pool_write_inline_kernel<1, true, N>), grid, block, 0, s, w);
            return hipGetLastError();
        };
        if (a.n_pages > kMaxInlineWrite) return hipErrorInvalidValue;
        if (a.n_pages <= 64) return go(std::integral_constant<int, 64>{});
        if (a.n_pages <= 256) return go(std::integral_constant<int, 256>{});
        return go(std::integral_constant<int, kMaxInlineWrite>{});
    }
    if (a.dtype == 0)
        hipLaunchKernelGGL((pool_write_kernel<0, false>), grid, block, 0, s, a);
    else if (!pairs)
        hipLaunchKernelGGL((pool_write_kernel<1, false>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((pool_write_kernel<1, true>), grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace hkv
