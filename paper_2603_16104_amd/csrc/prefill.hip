// Kernels of the 256-row attention tile (tile_body.h): suffix-only prefill (Section 5, "Token usage") and the
// decode work items shared by many query rows as a kernel of their own, for plans that run them next to
// the kernel of the other items on a second stream.
#include <hip/hip_ext.h>

#include "tile_body.h"

namespace hkv {

namespace {

using namespace tile;

template <bool DECODE, bool FP8>
__global__ __launch_bounds__(kThreads, 2) void attn_tile_kernel(TileArgs a) {
    __shared__ __attribute__((aligned(16))) char lds[kLdsBytes];
    if constexpr (!DECODE) {
        const PrefillTile t = static_cast<const PrefillTile *>(a.tiles)[blockIdx.x];
        if (t.n_q * (a.num_q_heads / a.pool.num_kv_heads) <= 64 && t.prefix_len + t.q_begin + t.n_q > kPrefillHalvesTokens) {
            body<false, false, false, true>(a, lds, (int)blockIdx.x, 1);
            return;
        }
    }
    body<DECODE, FP8>(a, lds, (int)blockIdx.x, (int)gridDim.x);
}

// Prefill tiles split along their keys: a persistent workgroup per compute unit runs an equal share of all key blocks.
// Bound by the matrix cores like the tile itself; a batch of fewer tiles than compute units (or a little more than a
// whole number of rounds) leaves the rest of the chip idle otherwise.  700 new tokens over 4096 cached ones, 88 tiles:
// 94.2 us a workgroup per tile (0.54 PFLOP/s), 60.4 us split, both kernels (0.84).
__global__ __launch_bounds__(kThreads, 2) void prefill_split_kernel(TileArgs a) {
    __shared__ __attribute__((aligned(16))) char lds[kLdsBytes];
    body<false, false, true>(a, lds, (int)blockIdx.x, 1);
}

// Combines the partials of the cut tiles: a workgroup per 32 rows of a tile, a wavefront per quarter of their 128 dims, in
// the accumulators' register order, so that every load is a whole KiB; log-sum-exp weights from the references and row sums.
// Bound by the partials' bytes once enough wavefronts have loads in flight: 88 tiles in 256 shares (45 MB)
// 12.4 -> 8.9 us (5 TB/s) against a wavefront per 32 whole rows; 64 new tokens over 8192 cached ones, 8 tiles of one
// 32-row part each in 256 shares, 53 -> 33 us with the tiles (32 by now).
__global__ __launch_bounds__(256) void prefill_merge_kernel(PrefillLaunch p) {
    const PrefillSplitTile st = p.split[blockIdx.x];
    const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
    const int rt = (int)blockIdx.y, quarter = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int G = p.num_q_heads / p.pool.num_kv_heads;
    const int r_tile = 32 * rt + n, tok = r_tile / G;
    if (rt == 0 && threadIdx.x == 0 && p.fallback_tiles) {
        int any = 0;
        for (int k = 0; k < st.n_parts; ++k) any |= p.part_bail[st.part0 + k];
        if (any) atomicAdd(p.fallback_tiles, 1u);
    }
    if (32 * rt / G >= st.t.n_q) return;  // (workgroup-uniform) no row of these exists
    const float *pd = p.part_data + (size_t)st.part0 * kSplitPartFloats;
    const float *pm = pd + 256 * kHeadDim + 64 * rt + n;
    float M = -INFINITY;
#pragma unroll 4
    for (int k = 0; k < st.n_parts; ++k) M = fmaxf(M, pm[k * kSplitPartFloats]);
    f32x4 acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    float L = 0.f;
#pragma unroll 4
    for (int k = 0; k < st.n_parts; ++k) {
        const float w = fast_exp2(pm[k * kSplitPartFloats] - M);  // (a row sees its own key at least: M is finite)
        L += w * pm[k * kSplitPartFloats + 32];
        const f32x4 *po = reinterpret_cast<const f32x4 *>(pd + k * kSplitPartFloats) + rt * (16 * 64) + quarter * (4 * 64) + lane;
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] += po[64 * i] * w;
    }
    if (tok >= st.t.n_q) return;
    const float inv = 1.0f / L;
    const uint32_t io_row = (uint32_t)(st.t.q_row0 + tok) * p.num_q_heads + st.t.kv_head * G + r_tile % G;
    uint16_t *op = static_cast<uint16_t *>(p.out) + (size_t)io_row * kHeadDim + 32 * quarter;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        u32x2 w;
        w[0] = pack_bf16(acc[i][0] * inv, acc[i][1] * inv);
        w[1] = pack_bf16(acc[i][2] * inv, acc[i][3] * inv);
        *reinterpret_cast<u32x2 *>(op + 8 * i + 4 * h) = w;
    }
    if (p.lse_out && quarter == 0 && h == 0) p.lse_out[io_row] = (M + fast_log2(L)) * kLn2;
}

}  // namespace

int prefill_tile_tokens(int group) { return 256 / group; }

hipError_t launch_prefill(const PrefillLaunch &p, hipStream_t s) {
    if (p.n_tiles <= 0) return hipSuccess;
    TileArgs a{};
    a.pool = p.pool;
    a.q = p.q;
    a.tiles = p.tiles;
    a.ids = p.block_table;
    a.n_tiles = p.n_tiles;
    a.num_q_heads = p.num_q_heads;
    a.scale = p.scale;
    a.out = p.out;
    a.lse_out = p.lse_out;
    a.fallback_tiles = p.fallback_tiles;
    if (p.n_workers > 0) {
        a.tiles = p.segments;
        a.seg_begin = p.seg_begin;
        a.part_data = p.part_data;
        a.part_bail = p.part_bail;
        hipLaunchKernelGGL(prefill_split_kernel, dim3(p.n_workers), dim3(kThreads), 0, s, a);
        if (p.n_split > 0) hipLaunchKernelGGL(prefill_merge_kernel, dim3(p.n_split, 8), dim3(256), 0, s, p);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((attn_tile_kernel<false, false>), dim3(p.n_tiles), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_decode_tiles(const DecodeTilesLaunch &d, hipStream_t s, hipEvent_t ev_begin, hipEvent_t ev_end) {
    if (d.n_items <= 0) return hipSuccess;
    if (d.n_workgroups <= 0 || (d.pool.dtype != 0 && d.pool.dtype != 1)) return hipErrorInvalidValue;
    TileArgs a{};
    a.pool = d.pool;
    a.q = d.q;
    a.tiles = d.items;
    a.ids = d.pages;
    a.n_tiles = d.n_items;
    a.num_q_heads = d.num_q_heads;
    a.scale = d.scale;
    a.node_req_idx = d.node_req_idx;
    a.o_parts = d.o_parts;
    a.lse_parts = d.lse_parts;
    a.max_parts = d.max_parts;
    a.down_parts = d.down_parts;
    a.q_rows = d.q_rows;
    const dim3 grid(d.n_workgroups < d.n_items ? d.n_workgroups : d.n_items);
    if (d.pool.dtype == 0)
        hipExtLaunchKernelGGL((attn_tile_kernel<true, false>), grid, dim3(kThreads), 0, s, ev_begin, ev_end, 0, a);
    else
        hipExtLaunchKernelGGL((attn_tile_kernel<true, true>), grid, dim3(kThreads), 0, s, ev_begin, ev_end, 0, a);
    return hipGetLastError();
}

}  // namespace hkv
