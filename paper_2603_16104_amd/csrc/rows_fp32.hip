// Full-precision path for fp32 pools: plain softmax attention of every query row over its request's
// block table, all arithmetic in fp32 on the vector ALUs (no matrix cores, no bf16 rounding anywhere),
// so that fp32 inputs meet the 1e-4 bound.  Nothing is shared between requests here: this path is for
// checking and for callers that need the precision.  (Same definition as everywhere: Section 2, "Scope":
// the result equals plain attention over the request's whole key/value sequence.)
//
// fp32 block format: K in 64-byte dimension chunks of 16 floats, chunk-major then slot
// ((d / 16) * 256 + slot * 16 + d % 16); V dimension-major (d * 16 + slot).
#include <algorithm>
#include <type_traits>

#include "hkv_device.h"

namespace hkv {

namespace {

// One workgroup per (query token, KV head, up to kRows of its query heads): its wavefronts take turns at steps of two
// pages (kRows = 4: of one) and combine in LDS.  Bound by the latency of a chain of steps per wavefront (K of the next step is
// requested behind the first product, V behind the second), then by K/V from L2: a compute unit takes in about 110 bytes per ns, so
// what counts is how many heads share a read.  Every load is one KiB a wavefront: lane = (slot, quarter of a 16-dimension chunk) for
// K, (dimension, quarter of the slots) for V, so a dot product is 32 multiply-adds in a lane and two adds over its quad.  A wavefront
// per (token, head) with a lane per key read 64-byte pieces, walked all keys alone and took 118 us for 16 requests x 32 heads over
// 1024 + 256 tokens on half of the chip, with three times the rounding error, the dot products being longer chains; two heads a
// workgroup take 18.2 us there (512 new tokens over 2048: 3.02 -> 0.77 ms).  Four heads and twice the rows: see row_heads_per_workgroup.
// SPLIT: a workgroup takes one of n_parts shares of its rows' steps and leaves its sums to rows_fp32_merge_kernel, so that few rows
// use the whole chip: those 16 requests 18.2 -> 16.8 us (two shares of four heads), 4 of them 17.4 -> 11.7, one over 4196 tokens 44.1 -> 16.1,
// 32 of 8 / 2 heads over 2348 25.9 -> 19.4.
constexpr int kRowWaves = 8;  // at most; fewer for short sequences (the launch decides)

__device__ __forceinline__ float quad_sum(float v) {
    v += dpp<kQuadXor1>(v);
    return v + dpp<kQuadXor2>(v);
}

template <int kRows, bool SPLIT>
__global__ __launch_bounds__(64 * kRowWaves, 2) void rows_fp32_kernel(RowsLaunch a) {
    static_assert(kRows == 1 || kRows == 2 || kRows == 4, "a lane of a quad stands for one row and page of a step");
    constexpr int kStepPages = kRows == 4 ? 1 : 2, kStepKeys = kStepPages * kPage;
    __shared__ float sP[kRowWaves][kRows][kStepKeys];
    __shared__ float sO[kRowWaves][kRows][kHeadDim];
    __shared__ float sM[kRowWaves][kRows], sL[kRowWaves][kRows];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int Hkv = a.pool.num_kv_heads, G = a.num_q_heads / Hkv;
    const int groups = kRows == 1 ? 1 : (G + kRows - 1) / kRows;  // (one row: for G = 1)
    const int per_group = kRows == 4 ? (G + groups - 1) / groups : kRows;
    const int kvh = (int)(blockIdx.x % Hkv);  // a head stays on its XCD where there are eight
    const int n_parts = SPLIT ? a.n_parts : 1, part = SPLIT ? (int)(blockIdx.x / Hkv) % n_parts : 0;
    const int rest = (int)(blockIdx.x / Hkv) / n_parts, h0 = kRows == 1 ? 0 : rest % groups * per_group, tq = kRows == 1 ? rest : rest / groups;
    const int len = a.row_len[tq];  // keys this query token sees
    const int32_t *bt = a.block_table + (size_t)a.row_req[tq] * a.max_pages;
    const float *K = static_cast<const float *>(a.pool.k_pages) + (size_t)kvh * kBlockElems + 4 * lane;
    const float *V = static_cast<const float *>(a.pool.v_pages) + (size_t)kvh * kBlockElems + 4 * lane;
    const size_t page_stride = (size_t)Hkv * kBlockElems;
    const int slot = lane >> 2, quarter = lane & 3, n_waves = (int)blockDim.x >> 6;
    // in a quad every lane owns one (page of the step, row): its exponentials and row sums
    const int own_page = kRows == 4 ? 0 : kRows == 2 ? quarter >> 1 : quarter & 1, own_row = kRows == 4 ? quarter : kRows == 2 ? quarter & 1 : 0;
    const bool counts = kRows > 1 || quarter < 2;  // (one row: the upper two lanes repeat the lower two)
    const float c = a.scale * kLog2e;

    f32x4 qf[kRows][8];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const float *qp = a.q + ((size_t)tq * a.num_q_heads + kvh * G + min(h0 + r, G - 1)) * kHeadDim + 4 * quarter;
#pragma unroll
        for (int i = 0; i < 8; ++i) qf[r][i] = *reinterpret_cast<const f32x4 *>(qp + 16 * i);
    }
    // (SPLIT: this workgroup's share of the steps, in whole ones)
    const int all_steps = (len + kStepKeys - 1) / kStepKeys;
    const int first_step = SPLIT ? (int)((int64_t)all_steps * part / n_parts) : 0, n_steps = SPLIT ? (int)((int64_t)all_steps * (part + 1) / n_parts) : all_steps;
    const int last_page = max(len - 1, 0) >> 4;
    f32x4 kf[kStepPages][8], vf[kStepPages][8];
    auto fetch = [&](f32x4 (&f)[kStepPages][8], const float *base, int step) {
#pragma unroll
        for (int g = 0; g < kStepPages; ++g) {
            const float *p = base + (size_t)bt[min(step * kStepPages + g, last_page)] * page_stride;
#pragma unroll
            for (int i = 0; i < 8; ++i) f[g][i] = *reinterpret_cast<const f32x4 *>(p + 256 * i);
        }
    };
    // Of the own row: running maximum (times scale * log2 e), this lane's share of the row sum.  It begins at the lowest finite
    // number: scores of -inf have weight 0 against that, not exp2(inf - inf), however many come first.
    constexpr float kLowest = -3.40282347e38f;
    float m, l;
    f32x4 acc[kRows][2];  // dims 16 i + slot of row r, this lane's quarter of the slots: element i % 4 of acc[r][i / 4]
    // A value whose weight underflows to zero takes no part, whatever it is (0 * inf would be NaN).  Asking for that at every
    // product would double the vector instructions, and infinities stay in a sum once they are there: a wavefront that ends
    // with one in its sums walks its keys a second time, asking.  (Two loops: one with a flag took 256 registers
    // instead of 241; 23 x 84 new tokens x 32 heads over 240, 753 -> 683 us.)
    auto walk = [&](auto careful_tag) {
        constexpr bool kCareful = decltype(careful_tag)::value;
        m = kLowest;
        l = 0.f;
#pragma unroll
        for (int r = 0; r < kRows; ++r) acc[r][0] = acc[r][1] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (first_step + wave < n_steps) {
            fetch(kf, K, first_step + wave);
            fetch(vf, V, first_step + wave);
        }
        for (int step = first_step + wave; step < n_steps; step += n_waves) {
            float s[kStepPages][kRows];
#pragma unroll
            for (int g = 0; g < kStepPages; ++g)
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    float dot = 0.f;
#pragma unroll
                    for (int i = 0; i < 8; ++i)
#pragma unroll
                        for (int j = 0; j < 4; ++j) dot = __builtin_fmaf(qf[r][i][j], kf[g][i][j], dot);
                    s[g][r] = quad_sum(dot);
                }
            __builtin_amdgcn_sched_barrier(0);
            fetch(kf, K, step + n_waves);  // the K registers are free (behind the last step: its page again, in bounds)
            __builtin_amdgcn_sched_barrier(0);
            float x = s[0][0];  // of the own row and page
#pragma unroll
            for (int g = 0; g < kStepPages; ++g)
#pragma unroll
                for (int r = 0; r < kRows; ++r)
                    if (g + r > 0) x = own_page == g && own_row == r ? s[g][r] : x;
            x = (step * kStepPages + own_page) * kPage + slot < len ? x * c : -INFINITY;
            float mx = fmaxf(x, dpp<kRor4>(x));  // over the lanes of the own row: slots ...
            mx = fmaxf(mx, dpp<kRor8>(mx));
            mx = rows_max(mx);
            if (kStepPages == 2) mx = fmaxf(mx, kRows == 2 ? dpp<kQuadXor2>(mx) : dpp<kQuadXor1>(mx));  // ... and pages
            const float m_new = fmaxf(m, mx);
            const float alpha = fast_exp2(m - m_new);
            const float p = fast_exp2(x - m_new);
            l = l * alpha + p;
            m = m_new;
            if (counts) sP[wave][own_row][own_page * kPage + slot] = p;
            __builtin_amdgcn_wave_barrier();  // (LDS operations of one wavefront execute in order)
            const bool tail = (step + 1) * kStepKeys > len;
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                // the row's factor from its lane of the quad
                const float al = kRows == 1 ? alpha : r == 0 ? dpp<0x00>(alpha) : r == 1 ? dpp<0x55>(alpha) : r == 2 ? dpp<0xAA>(alpha) : dpp<0xFF>(alpha);
                acc[r][0] *= al;
                acc[r][1] *= al;
                if (kCareful && al == 0.f) acc[r][0] = acc[r][1] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int g = 0; g < kStepPages; ++g) {
                if (tail) {  // slots past the sequence end may hold anything (NaN included)
                    const int left = len - (step * kStepPages + g) * kPage - 4 * quarter;
#pragma unroll
                    for (int i = 0; i < 8; ++i)
#pragma unroll
                        for (int j = 0; j < 4; ++j) vf[g][i][j] = j < left ? vf[g][i][j] : 0.f;
                }
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    const f32x4 pr = *reinterpret_cast<const f32x4 *>(&sP[wave][r][g * kPage + 4 * quarter]);
                    if constexpr (kCareful) {
#pragma unroll
                        for (int i = 0; i < 8; ++i)
#pragma unroll
                            for (int j = 0; j < 4; ++j)
                                if (pr[j] != 0.f) acc[r][i >> 2][i & 3] = __builtin_fmaf(pr[j], vf[g][i][j], acc[r][i >> 2][i & 3]);
                    } else {
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            float o = acc[r][i >> 2][i & 3];
#pragma unroll
                            for (int j = 0; j < 4; ++j) o = __builtin_fmaf(pr[j], vf[g][i][j], o);
                            acc[r][i >> 2][i & 3] = o;
                        }
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            fetch(vf, V, step + n_waves);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_wave_barrier();
        }
    };
    walk(std::false_type{});
    float zero = 0.f;  // NaN if any sum is not finite
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int i = 0; i < 8; ++i) zero = __builtin_fmaf(acc[r][i >> 2][i & 3], 0.f, zero);
    if (__builtin_amdgcn_ballot_w64(zero != 0.f)) walk(std::true_type{});
    // the own row's sum over its lanes, the dims over the quads; then the wavefronts
    float lt = l + dpp<kRor4>(l);
    lt += dpp<kRor8>(lt);
    lt = rows_sum(lt);
    if (kStepPages == 2) lt += kRows == 2 ? dpp<kQuadXor2>(lt) : dpp<kQuadXor1>(lt);
    if (lane < kRows) {  // lane r owns row r
        sM[wave][lane] = m;
        sL[wave][lane] = lt;
    }
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float o = quad_sum(acc[r][i >> 2][i & 3]);
            if (quarter == (i & 3)) sO[wave][r][16 * i + slot] = o;
        }
    __syncthreads();
    for (int t = threadIdx.x; t < kRows * kHeadDim; t += blockDim.x) {
        const int r = t / kHeadDim, d = t % kHeadDim;
        if (r >= per_group || h0 + r >= G) return;
        float M = -INFINITY;
        for (int w = 0; w < n_waves; ++w) M = fmaxf(M, sM[w][r]);
        float L = 0.f, out = 0.f;
        for (int w = 0; w < n_waves; ++w) {
            const float f = fast_exp2(sM[w][r] - M);
            L = __builtin_fmaf(sL[w][r], f, L);
            const float with = __builtin_fmaf(sO[w][r][d], f, out);
            out = f != 0.f ? with : out;
        }
        const size_t row = (size_t)tq * a.num_q_heads + kvh * G + h0 + r;
        if constexpr (SPLIT) {  // for rows_fp32_merge_kernel
            float *pd = a.part_data + (row * n_parts + part) * kRowPartFloats;
            pd[d] = out;
            if (d == 0) {
                pd[kHeadDim] = M;
                pd[kHeadDim + 1] = L;
            }
            continue;
        }
        // a row without keys gives out = 0, lse = -inf; one whose scores hold a NaN or +inf, or only -inf, gives NaN
        a.out[row * kHeadDim + d] = L > 0.f ? out / L : len > 0 ? __builtin_nanf("") : 0.f;
        if (a.lse_out && d == 0) a.lse_out[row] = L > 0.f ? (M + fast_log2(L)) * kLn2 : -INFINITY;
    }
}

// Combines the parts of a row that SPLIT leaves: a wavefront per row.  The same sums, in the same manner, as those over the
// wavefronts of a workgroup.
__global__ __launch_bounds__(256) void rows_fp32_merge_kernel(RowsLaunch a) {
    const int row = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63, n = a.n_parts;
    if (row >= a.n_q_tokens * a.num_q_heads) return;
    const int len = a.row_len[row / a.num_q_heads];
    const float *pd = a.part_data + (size_t)row * n * kRowPartFloats;
    const float m = lane < n ? pd[lane * kRowPartFloats + kHeadDim] : -INFINITY, l = lane < n ? pd[lane * kRowPartFloats + kHeadDim + 1] : 0.f;  // (n <= kMaxRowParts)
    float M = m;
#pragma unroll
    for (int sh = 1; sh < 64; sh <<= 1) M = fmaxf(M, __shfl_xor(M, sh));
    const float f = fast_exp2(m - M);
    float L = 0.f, o0 = 0.f, o1 = 0.f;
    for (int k0 = 0; k0 < n; k0 += 8) {  // (shares beyond the last have weight 0)
        float2 o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = *reinterpret_cast<const float2 *>(pd + min(k0 + j, n - 1) * kRowPartFloats + 2 * lane);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float fk = __shfl(f, k0 + j);
            L = __builtin_fmaf(__shfl(l, k0 + j), fk, L);
            o0 = fk != 0.f ? __builtin_fmaf(o[j].x, fk, o0) : o0;
            o1 = fk != 0.f ? __builtin_fmaf(o[j].y, fk, o1) : o1;
        }
    }
    const float none = len > 0 ? __builtin_nanf("") : 0.f;
    *reinterpret_cast<float2 *>(a.out + (size_t)row * kHeadDim + 2 * lane) = L > 0.f ? make_float2(o0 / L, o1 / L) : make_float2(none, none);
    if (a.lse_out && lane == 0) a.lse_out[row] = L > 0.f ? (M + fast_log2(L)) * kLn2 : -INFINITY;
}

// fp32 source tokens -> fp32 block format, one thread per element
__global__ __launch_bounds__(256) void pool_write_fp32_kernel(PoolWriteLaunch a) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    const long n = (long)a.n_tokens * a.num_kv_heads * kHeadDim;
    if (i >= n) return;
    const int d = (int)(i % kHeadDim), h = (int)((i / kHeadDim) % a.num_kv_heads), t = (int)(i / ((long)kHeadDim * a.num_kv_heads));
    const int pos = a.first_slot + t, page = a.page_ids[pos >> 4], slot = pos & 15;
    const size_t blk = ((size_t)page * a.num_kv_heads + h) * kBlockElems;
    static_cast<float *>(a.k_pages)[blk + (d >> 4) * 256 + slot * 16 + (d & 15)] = static_cast<const float *>(a.k_src)[i];
    static_cast<float *>(a.v_pages)[blk + d * 16 + slot] = static_cast<const float *>(a.v_src)[i];
}

}  // namespace

hipError_t launch_rows_fp32(const RowsLaunch &a, hipStream_t s) {
    const int Hkv = a.pool.num_kv_heads, G = a.num_q_heads / Hkv;
    const bool split = a.n_parts > 1;
    if (split && (!a.part_data || a.n_parts > kMaxRowParts)) return hipErrorInvalidValue;
    // a step is 32 keys (four heads: 16): sequences that never reach four steps a wavefront would pay for wavefronts without one (128 query
    // tokens of 17 to 32 keys, 32 heads: 24.2 us with eight, 12.5 us with two; a share has about 128 keys and more of the longest row, and what there is of the others)
    const int waves = split || a.max_pages > 16 ? kRowWaves : a.max_pages > 8 ? 4 : 2;
    const int rows = row_heads_per_workgroup(a.n_q_tokens, Hkv, G, a.max_pages, split);
    const size_t per_token = (size_t)Hkv * ((G + rows - 1) / rows) * std::max(1, a.n_parts);
    const size_t most = std::max<size_t>(1, ((size_t)1 << 31) / (per_token * 64 * waves));  // query tokens of a launch: below 2^32 threads
    for (size_t t0 = 0; t0 < (size_t)std::max(a.n_q_tokens, 0); t0 += most) {
        RowsLaunch b = a;
        b.n_q_tokens = (int32_t)std::min(most, (size_t)a.n_q_tokens - t0);
        b.q += t0 * a.num_q_heads * kHeadDim;
        b.out += t0 * a.num_q_heads * kHeadDim;
        if (b.lse_out) b.lse_out += t0 * a.num_q_heads;
        b.row_req += t0;
        b.row_len += t0;
        if (split) b.part_data += t0 * a.num_q_heads * a.n_parts * kRowPartFloats;
        const dim3 grid((unsigned)(b.n_q_tokens * per_token)), block(64 * waves);
        auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, s, b); };
        if (split)
            rows == 1 ? go(rows_fp32_kernel<1, true>) : rows == 2 ? go(rows_fp32_kernel<2, true>) : go(rows_fp32_kernel<4, true>);
        else
            rows == 1 ? go(rows_fp32_kernel<1, false>) : rows == 2 ? go(rows_fp32_kernel<2, false>) : go(rows_fp32_kernel<4, false>);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    if (split && a.n_q_tokens > 0) {
        hipLaunchKernelGGL(rows_fp32_merge_kernel, dim3((unsigned)((a.n_q_tokens * a.num_q_heads + 3) / 4)), dim3(256), 0, s, a);
        return hipGetLastError();
    }
    return hipSuccess;
}

hipError_t launch_pool_write_fp32(const PoolWriteLaunch &a, hipStream_t s) {
    const long n = (long)a.n_tokens * a.num_kv_heads * kHeadDim;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(pool_write_fp32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace hkv
