// Log-sum-exp combine of partial attention results (one wavefront per output row).
//   lse = ln sum_n exp(lse_n),  out = sum_n exp(lse_n - lse) * o_n
// A partial with lse = -inf is skipped without reading its o (which may hold anything); a row
// without finite partials gives out = 0, lse = -inf.
#include <hip/hip_ext.h>

#include <type_traits>

#include "hkv_device.h"

namespace hkv {

namespace {

constexpr int kRowsPerBlock = 4;

template <int OUT_DT>
__global__ __launch_bounds__(64 * kRowsPerBlock) void lse_merge_kernel(const float *__restrict__ o_parts,
                                                                        const float *__restrict__ lse_parts,
                                                                        const int32_t *__restrict__ row_indptr,
                                                                        const int32_t *__restrict__ part_idx,
                                                                        int32_t n_rows, void *__restrict__ out,
                                                                        float *__restrict__ lse_out) {
    const int row = blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= n_rows) return;
    const int beg = row_indptr[row], end = row_indptr[row + 1];
    float M = -INFINITY;
    for (int k = beg; k < end; ++k) M = fmaxf(M, lse_parts[part_idx[k]]);
    float acc0 = 0.f, acc1 = 0.f, z = 0.f;
    if (M != -INFINITY) {
        for (int k = beg; k < end; ++k) {
            const int n = part_idx[k];
            const float ls = lse_parts[n];
            if (ls == -INFINITY) continue;
            const float w = fast_exp2((ls - M) * kLog2e);
            const float2 o = *reinterpret_cast<const float2 *>(o_parts + (size_t)n * kHeadDim + 2 * lane);
            z += w;
            acc0 = __builtin_fmaf(w, o.x, acc0);
            acc1 = __builtin_fmaf(w, o.y, acc1);
        }
        const float inv = 1.0f / z;
        acc0 *= inv;
        acc1 *= inv;
    }
    if (OUT_DT == 0) {
        reinterpret_cast<uint32_t *>(out)[(size_t)row * (kHeadDim / 2) + lane] = pack_bf16(acc0, acc1);
    } else {
        reinterpret_cast<float2 *>(out)[(size_t)row * (kHeadDim / 2) + lane] = make_float2(acc0, acc1);
    }
    if (lse_out && lane == 0) lse_out[row] = (M == -INFINITY) ? -INFINITY : M + fast_log2(z) * kLn2;
}

// Dense variant: row i owns partials i*max_parts + k, k < part_count[i / rows_per_count].  Up to 8 partials: half a wavefront
// per row (32 lanes x 4 dims); the partials and their lse values are requested together, so a row costs one memory round
// trip (kUnroll: the number of slots, 2, 3, 4, 6 or 8).
constexpr int kDenseRowsPerBlock = 8;
constexpr int kManyRows = 16384;  // from here on a half wavefront merges four rows (fp16 partials: lse_merge_wide_kernel)

// four consecutive values of a partial, as floats
template <bool PB16>
__device__ __forceinline__ f32x4 load_part4(const void *o_parts, size_t elem) {
    if constexpr (PB16) {  // fp16; the caller applies the partial's factor
        const u32x2 w = *reinterpret_cast<const u32x2 *>(static_cast<const uint16_t *>(o_parts) + elem);
        const uint32_t w0 = w[0], w1 = w[1];  // (a bit cast straight from a vector element reads element 0 for both)
        const f16x2 a = __builtin_bit_cast(f16x2, w0), b = __builtin_bit_cast(f16x2, w1);
        return f32x4{(float)a[0], (float)a[1], (float)b[0], (float)b[1]};
    } else {
        return *reinterpret_cast<const f32x4 *>(static_cast<const float *>(o_parts) + elem);
    }
}

template <int OUT_DT, int kUnroll, bool PB16>
__device__ __forceinline__ void merge_dense_row(const void *__restrict__ o_parts, const float *__restrict__ lse_parts,
                                                const int32_t *__restrict__ part_count, int32_t rows_per_count,
                                                int32_t max_parts, int row, int l, void *__restrict__ out,
                                                float *__restrict__ lse_out, const int32_t *__restrict__ out_rows,
                                                const float *__restrict__ down_parts) {
    const int cnt = min(part_count[row / rows_per_count], max_parts);
    const size_t base = (size_t)row * max_parts;
    const float *lp = lse_parts + base;
    const float *dp = PB16 ? down_parts + base : nullptr;  // fp16 partials: the factor each one is to be multiplied by
    const size_t o0 = base * kHeadDim + 4 * l;  // element index of this lane's four dims in slot 0
    // All slots are requested before the count is known (slots k < max_parts exist for every row; what an unused one holds
    // is never looked at), so the count, the lse values and the partials travel in one round trip instead of two.
    float ls[kUnroll], ds[kUnroll];
    f32x4 ov[kUnroll];
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) {
        const int kc = min(k, max_parts - 1);
        ls[k] = lp[kc];
        ds[k] = PB16 ? dp[kc] : 1.0f;
        ov[k] = load_part4<PB16>(o_parts, o0 + (size_t)kc * kHeadDim);
    }
#pragma unroll
    for (int k = 0; k < kUnroll; ++k)
        if (k >= cnt) ls[k] = -INFINITY;
    float M = -INFINITY;
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) M = fmaxf(M, ls[k]);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float z = 0.f;
    if (M != -INFINITY) {
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
            if (ls[k] != -INFINITY) {  // an empty partial may hold anything in o
                const float w = fast_exp2((ls[k] - M) * kLog2e);
                z += w;
                acc += ov[k] * (w * ds[k]);
            }
        }
        acc *= 1.0f / z;
    }
    const size_t dst = out_rows ? (size_t)out_rows[row / rows_per_count] * rows_per_count + row % rows_per_count : (size_t)row;
    if (OUT_DT == 0) {
        u32x2 w;
        w[0] = pack_bf16(acc[0], acc[1]);
        w[1] = pack_bf16(acc[2], acc[3]);
        reinterpret_cast<u32x2 *>(out)[dst * (kHeadDim / 4) + l] = w;
    } else {
        reinterpret_cast<f32x4 *>(out)[dst * (kHeadDim / 4) + l] = acc;
    }
    if (lse_out && l == 0) lse_out[dst] = (M == -INFINITY) ? -INFINITY : M + fast_log2(z) * kLn2;
}

// kRowsPerLane rows per half wavefront (rows row0, row0 + stride, ...): large batches run four, whose loads the
// compiler issues together, on a quarter of the workgroups.
template <int OUT_DT, int kUnroll, bool PB16, int kRowsPerLane>
__global__ __launch_bounds__(32 * kDenseRowsPerBlock) void lse_merge_dense_kernel(
    const void *__restrict__ o_parts, const float *__restrict__ lse_parts, const int32_t *__restrict__ part_count,
    int32_t rows_per_count, int32_t max_parts, int32_t n_rows, void *__restrict__ out, float *__restrict__ lse_out,
    const int32_t *__restrict__ out_rows, const float *__restrict__ down_parts) {
    const int row0 = (blockIdx.x * kRowsPerLane) * kDenseRowsPerBlock + (threadIdx.x >> 5);
    const int l = threadIdx.x & 31;
#pragma unroll
    for (int r = 0; r < kRowsPerLane; ++r) {
        const int row = row0 + r * kDenseRowsPerBlock;
        if (row < n_rows)
            merge_dense_row<OUT_DT, kUnroll, PB16>(o_parts, lse_parts, part_count, rows_per_count, max_parts, row, l, out,
                                                   lse_out, out_rows, down_parts);
    }
}

template <bool PB16>
__device__ __forceinline__ void load_part8(const void *o_parts, size_t elem, f32x4 &lo, f32x4 &hi) {
    if constexpr (PB16) {
        const u32x4 w = *reinterpret_cast<const u32x4 *>(static_cast<const uint16_t *>(o_parts) + elem);
        const uint32_t w0 = w[0], w1 = w[1], w2 = w[2], w3 = w[3];
        const f16x2 a = __builtin_bit_cast(f16x2, w0), b = __builtin_bit_cast(f16x2, w1), c = __builtin_bit_cast(f16x2, w2), d = __builtin_bit_cast(f16x2, w3);
        lo = f32x4{(float)a[0], (float)a[1], (float)b[0], (float)b[1]};
        hi = f32x4{(float)c[0], (float)c[1], (float)d[0], (float)d[1]};
    } else {
        lo = reinterpret_cast<const f32x4 *>(static_cast<const float *>(o_parts) + elem)[0];
        hi = reinterpret_cast<const f32x4 *>(static_cast<const float *>(o_parts) + elem)[1];
    }
}

// Decode steps of kManyRows rows and more: a quarter of a wavefront per row, 16 bytes a lane, so that one load takes a KiB.  Bound by the
// partials' bytes (from L2 and the last-level cache, 5 to 6 TB/s).  Half a wavefront with 8 bytes a lane, four rows of it in flight, took 8.2 us for 43008
// rows x 2 (this: 6.9), 7.2 for 32768 x 2 (5.7), 6.6 for 16384 x 3 (4.7); with two rows in flight this takes 0.1 to 0.4 more, and below
// 16384 rows the two forms are within 0.2 of each other either way.
template <int kUnroll>
__global__ __launch_bounds__(256) void lse_merge_wide_kernel(const uint16_t *__restrict__ o_parts, const float *__restrict__ lse_parts,
                                                             const int32_t *__restrict__ part_count, int32_t rows_per_count, int32_t max_parts,
                                                             int32_t n_rows, void *__restrict__ out, float *__restrict__ lse_out,
                                                             const int32_t *__restrict__ out_rows, const float *__restrict__ down_parts) {
    const int row = (int)blockIdx.x * 16 + (int)(threadIdx.x >> 4), l = threadIdx.x & 15;
    if (row >= n_rows) return;
    const int cnt = min(part_count[row / rows_per_count], max_parts);
    const size_t base = (size_t)row * max_parts;
    // (all slots requested before the count is known, as in merge_dense_row)
    float ls[kUnroll], ds[kUnroll];
    f32x4 lo[kUnroll], hi[kUnroll];
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) {
        const int kc = min(k, max_parts - 1);
        ls[k] = lse_parts[base + kc];
        ds[k] = down_parts[base + kc];
        load_part8<true>(o_parts, (base + kc) * kHeadDim + 8 * l, lo[k], hi[k]);
    }
    float M = -INFINITY;
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) {
        if (k >= cnt) ls[k] = -INFINITY;
        M = fmaxf(M, ls[k]);
    }
    f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0;
    float z = 0.f;
    if (M != -INFINITY) {
#pragma unroll
        for (int k = 0; k < kUnroll; ++k)
            if (ls[k] != -INFINITY) {  // an empty partial may hold anything in o
                const float w = fast_exp2((ls[k] - M) * kLog2e), wd = w * ds[k];
                z += w;
                a0 += lo[k] * wd;
                a1 += hi[k] * wd;
            }
        const float inv = 1.0f / z;
        a0 *= inv;
        a1 *= inv;
    }
    const size_t dst = out_rows ? (size_t)out_rows[row / rows_per_count] * rows_per_count + row % rows_per_count : (size_t)row;
    reinterpret_cast<u32x4 *>(out)[dst * (kHeadDim / 8) + l] = u32x4{pack_bf16(a0[0], a0[1]), pack_bf16(a0[2], a0[3]), pack_bf16(a1[0], a1[1]), pack_bf16(a1[2], a1[3])};
    if (lse_out && l == 0) lse_out[dst] = (M == -INFINITY) ? -INFINITY : M + fast_log2(z) * kLn2;
}

// Rows of many partials: a wavefront per row, whose four rows of 16 lanes (8 dims a lane) take every fourth partial each, 4 * U
// of them in flight at once.  Bound by latency: half a wavefront per row, with 16 partials at once and the others one after
// the other, took 3.2 us for 512 rows x 9 (this: 2.6), 5.3 for 24 (3.1), 12.2 for 48 (3.8), 13.2 for 2048 rows x 32 (4.5); from
// some 8192 rows on both are bound by the partials' bytes (16 384 x 24: 34 / 30).  Below 9 partials half a wavefront per row is the
// faster form (512 x 8: 2.69 against 2.71 us, 2048 x 8: 2.85 against 3.08).
template <int OUT_DT, int U, bool PB16>
__global__ __launch_bounds__(64 * kRowsPerBlock) void lse_merge_deep_kernel(
    const void *__restrict__ o_parts, const float *__restrict__ lse_parts, const int32_t *__restrict__ part_count,
    int32_t rows_per_count, int32_t max_parts, int32_t n_rows, void *__restrict__ out, float *__restrict__ lse_out,
    const int32_t *__restrict__ out_rows, const float *__restrict__ down_parts) {
    const int row = blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
    if (row >= n_rows) return;
    const int lane = threadIdx.x & 63, sub = lane >> 4, l = lane & 15;
    const size_t base = (size_t)row * max_parts;
    const float *lp = lse_parts + base;
    // Up to 16 slots are requested before the count is known (slots below max_parts exist for every row; what an unused one holds
    // is never looked at).  With more of them most may be unused, and the count comes first.
    const int cnt = min(part_count[row / rows_per_count], max_parts);
    const int last = U <= 4 ? max_parts - 1 : max(cnt - 1, 0);
    float ls[U], ds[U];
    f32x4 lo[U], hi[U];
    auto request = [&](int k0) {
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int k = min(k0 + 4 * j + sub, last);
            ls[j] = lp[k];
            ds[j] = PB16 ? down_parts[base + k] : 1.0f;
            load_part8<PB16>(o_parts, (base + k) * kHeadDim + 8 * l, lo[j], hi[j]);
        }
    };
    float M = lp[min(lane, last)];
    request(0);
    if (lane >= cnt) M = -INFINITY;
    for (int k = 64 + lane; k < cnt; k += 64) M = fmaxf(M, lp[k]);
    M = fmaxf(M, dpp<kQuadXor1>(M));
    M = fmaxf(M, dpp<kQuadXor2>(M));
    M = fmaxf(M, dpp<kRor4>(M));
    M = fmaxf(M, dpp<kRor8>(M));
    M = rows_max(M);
    f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = {0.f, 0.f, 0.f, 0.f};
    float z = 0.f;
    if (M != -INFINITY) {
        for (int k0 = 0;;) {
#pragma unroll
            for (int j = 0; j < U; ++j)
                if (k0 + 4 * j + sub < cnt && ls[j] != -INFINITY) {  // an empty partial may hold anything in o
                    const float w = fast_exp2((ls[j] - M) * kLog2e), wd = w * ds[j];
                    z += w;
                    a0 += lo[j] * wd;
                    a1 += hi[j] * wd;
                }
            k0 += 4 * U;
            if (k0 >= cnt) break;
            request(k0);
        }
        z = rows_sum(z);
        const float inv = 1.0f / z;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a0[i] = rows_sum(a0[i]) * inv;
            a1[i] = rows_sum(a1[i]) * inv;
        }
    }
    const size_t dst = out_rows ? (size_t)out_rows[row / rows_per_count] * rows_per_count + row % rows_per_count : (size_t)row;
    if (sub == 0) {
        if (OUT_DT == 0) {
            reinterpret_cast<u32x4 *>(out)[dst * (kHeadDim / 8) + l] = u32x4{pack_bf16(a0[0], a0[1]), pack_bf16(a0[2], a0[3]), pack_bf16(a1[0], a1[1]), pack_bf16(a1[2], a1[3])};
        } else {
            reinterpret_cast<f32x4 *>(out)[dst * (kHeadDim / 4) + 2 * l] = a0;
            reinterpret_cast<f32x4 *>(out)[dst * (kHeadDim / 4) + 2 * l + 1] = a1;
        }
        if (lse_out && l == 0) lse_out[dst] = (M == -INFINITY) ? -INFINITY : M + fast_log2(z) * kLn2;
    }
}

}  // namespace

hipError_t launch_lse_merge_dense(const void *o_parts, const float *lse_parts, const int32_t *part_count,
                                  int32_t rows_per_count, int32_t max_parts, int32_t n_rows, void *out,
                                  int32_t out_dtype, float *lse_out, hipStream_t s, hipEvent_t ev_begin,
                                  hipEvent_t ev_end, const int32_t *out_rows, const float *down_parts) {
    if (n_rows <= 0) return hipSuccess;
    if (down_parts && out_dtype != 0) return hipErrorInvalidValue;  // fp16 partials are a decode step's, whose results are bf16
    const bool many = n_rows >= kManyRows;
    const int per_block = kDenseRowsPerBlock * (many ? 4 : 1);
    dim3 grid((n_rows + per_block - 1) / per_block), block(32 * kDenseRowsPerBlock);
    auto go = [&](auto kernel) {
        hipExtLaunchKernelGGL(kernel, grid, block, 0, s, ev_begin, ev_end, 0, o_parts, lse_parts, part_count,
                              rows_per_count, max_parts, n_rows, out, lse_out, out_rows, down_parts);
    };
    if (max_parts > 8) {
        const dim3 deep_grid((n_rows + kRowsPerBlock - 1) / kRowsPerBlock), deep_block(64 * kRowsPerBlock);
        auto deep = [&](auto kernel) {
            hipExtLaunchKernelGGL(kernel, deep_grid, deep_block, 0, s, ev_begin, ev_end, 0, o_parts, lse_parts, part_count,
                                  rows_per_count, max_parts, n_rows, out, lse_out, out_rows, down_parts);
        };
        auto of = [&](auto unroll, auto pb16) {
            constexpr int U = decltype(unroll)::value;
            constexpr bool PB = decltype(pb16)::value;
            if constexpr (PB)
                deep(lse_merge_deep_kernel<0, U, true>);
            else
                out_dtype == 0 ? deep(lse_merge_deep_kernel<0, U, false>) : deep(lse_merge_deep_kernel<2, U, false>);
        };
        if (max_parts <= 16)
            down_parts ? of(std::integral_constant<int, 4>{}, std::true_type{}) : of(std::integral_constant<int, 4>{}, std::false_type{});
        else
            down_parts ? of(std::integral_constant<int, 8>{}, std::true_type{}) : of(std::integral_constant<int, 8>{}, std::false_type{});
        return hipGetLastError();
    }
    if (down_parts && many) {
        auto wide = [&](auto unroll) {
            hipExtLaunchKernelGGL(lse_merge_wide_kernel<decltype(unroll)::value>, dim3((n_rows + 15) / 16), dim3(256), 0, s, ev_begin, ev_end, 0,
                                  static_cast<const uint16_t *>(o_parts), lse_parts, part_count, rows_per_count, max_parts, n_rows, out, lse_out, out_rows, down_parts);
        };
        if (max_parts <= 2) wide(std::integral_constant<int, 2>{});
        else if (max_parts == 3) wide(std::integral_constant<int, 3>{});
        else if (max_parts == 4) wide(std::integral_constant<int, 4>{});
        else if (max_parts <= 6) wide(std::integral_constant<int, 6>{});
        else wide(std::integral_constant<int, 8>{});
        return hipGetLastError();
    }
    auto pick = [&](auto pb16) {
        constexpr bool PB = decltype(pb16)::value;
        auto of = [&](auto unroll) {
            constexpr int U = decltype(unroll)::value;
            if constexpr (PB)
                go(lse_merge_dense_kernel<0, U, true, 1>);
            else if (many)
                out_dtype == 0 ? go(lse_merge_dense_kernel<0, U, false, 4>) : go(lse_merge_dense_kernel<2, U, false, 4>);
            else
                out_dtype == 0 ? go(lse_merge_dense_kernel<0, U, false, 1>) : go(lse_merge_dense_kernel<2, U, false, 1>);
        };
        if (max_parts <= 2) return of(std::integral_constant<int, 2>{});
        if (max_parts == 3) return of(std::integral_constant<int, 3>{});
        if (max_parts == 4) return of(std::integral_constant<int, 4>{});
        if (max_parts <= 6) return of(std::integral_constant<int, 6>{});
        of(std::integral_constant<int, 8>{});
    };
    if (down_parts)
        pick(std::true_type{});
    else
        pick(std::false_type{});
    return hipGetLastError();
}

hipError_t launch_lse_merge(const float *o_parts, const float *lse_parts, const int32_t *row_indptr,
                            const int32_t *part_idx, int32_t n_rows, void *out, int32_t out_dtype, float *lse_out,
                            hipStream_t s) {
    if (n_rows <= 0) return hipSuccess;
    dim3 grid((n_rows + kRowsPerBlock - 1) / kRowsPerBlock), block(64 * kRowsPerBlock);
    if (out_dtype == 0)
        hipLaunchKernelGGL(lse_merge_kernel<0>, grid, block, 0, s, o_parts, lse_parts, row_indptr, part_idx, n_rows,
                           out, lse_out);
    else
        hipLaunchKernelGGL(lse_merge_kernel<2>, grid, block, 0, s, o_parts, lse_parts, row_indptr, part_idx, n_rows,
                           out, lse_out);
    return hipGetLastError();
}

}  // namespace hkv
