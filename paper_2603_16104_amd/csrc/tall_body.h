// Decode items shared by 65 to 128 query rows of a bf16 pool (device code, called by rows_body.h): one workgroup of four
// wavefronts applies a chunk of a prefix-tree node to up to four 32-row tiles, a wavefront each over all tokens.  (Shared prefix KV
// computed once and reused by every call below it: Section 5, "Proactive Cache Management".)
//
// Matrix-core mapping, LDS image and ring as in shared_body.h.  What bounds it: vector and matrix instructions together.  A block of
// 64 tokens takes a wavefront 32 matrix instructions (1024 cycles) and about 270 vector ones (32 exponentials at 8 cycles, 64
// products where the reference moves); two wavefronts of a SIMD fill each other's gaps in part.  So the products are interleaved
// with the exponentials (ten pairs beside K Q^T, six and the next block's maxima beside V P^T), and the stretch that holds matrix
// instructions runs at a higher wave priority than the reference and its rescaling, so that of two wavefronts one is
// in either (a block 1.40 -> 1.27 us alone, 2.05 -> 1.90 two workgroups on a compute unit).  Measured over 2048 rows below 4096 more
// tokens: 1.05 to 1.1 PFLOP/s, 64-row items of shared_body.h 0.85, 16-row tiles, three workgroups on a compute unit, 0.75; K and V
// come from L2 once per 128 rows instead of 64.  64 requests x 21 drafted tokens x 32 heads over 2048 + 512: step 107.1 -> 89.8 us.
// Tried: P(j) kept for the next phase, so that all three streams overlap (102 registers spilled); four operands on their way
// from LDS instead of eight (the same time).
//
// The softmax reference is the running maximum, taken per block, and begins anew every 256 tokens, 2^4 below the row's largest so
// far: the maximum is the one weight that bf16 holds exactly and the next ones lie just below a power of two, where its rounding
// is finest.  Error against 64 bits over 2048 + 512 tokens: 0.00216; anew every 512 tokens 0.00220, never 0.00223; 16-row
// tiles in chunks of 512 0.00219.
#pragma once
#include "hkv_device.h"
#include "shared_body.h"

namespace hkv {

namespace tall {

using shared::halves_max;
using shared::halves_sum;
using shared::kBlockTokens;
using shared::wait_slots_in_flight;

constexpr int kAnewBlocks = 4;  // after so many blocks a reference begins anew

__device__ __forceinline__ void body(const DecodeLaunch &a, const DecodeItem &it, char *smem, const int wave, const int lane) {
    constexpr int kPageBytes = kBlockElems * 2;
    constexpr int kSlotBytes = 4 * kPageBytes;
    constexpr int kLoads = kPageBytes / 1024;       // LDS-direct loads per wavefront and half-block (wavefront w: page w)
    const int Hkv = a.pool.num_kv_heads, G = a.num_q_heads / Hkv;
    const int rows = it.n_req * G;
    const int n = lane & 31, h = lane >> 5;
    const bool active = 32 * wave < rows;           // wavefront-uniform
    const float c = a.scale * kLog2e;
    const int n_blk = (it.n_tokens + kBlockTokens - 1) / kBlockTokens;
    const int last_page = (it.n_tokens - 1) >> 4;
    const uint32_t page_stride = (uint32_t)Hkv * kPageBytes;
    const char *kbase = static_cast<const char *>(a.pool.k_pages) + (size_t)it.kv_head * kPageBytes;
    const char *vbase = static_cast<const char *>(a.pool.v_pages) + (size_t)it.kv_head * kPageBytes;

    const int32_t *ids = a.pages + it.page_off;
    // (ids and rows in one round trip, what stands behind the first requests in the next one; lane b holds page 4 b + wave, the one this
    // wavefront fetches in block b)
    const int id_lane = ids[min(4 * lane + wave, last_page)];
    const int row = 32 * wave + n, rowc = min(row, rows - 1);
    const int req = a.node_req_idx[it.req_off + rowc / G];

    const int l_slot = lane >> 2;
    const uint32_t k_src = (uint32_t)(l_slot * 64 + (((lane & 3) ^ ((wave & 1) | ((((l_slot >> 1) ^ (l_slot >> 2)) & 1) << 1))) << 4));
    const uint32_t v_src = (uint32_t)((lane >> 1) * 32 + (((lane & 1) ^ (((lane >> 3) ^ (lane >> 4)) & 1)) << 4));
    const int n_slots = min(a.n_stages * (16384 / kSlotBytes), 9);
    const int n_req = 2 * n_blk;
    int issued = 0, put = 0;
    const uint32_t lds0 = lds_address(smem) + wave * kPageBytes;
    auto request = [&]() {  // the next half-block: number r is K (r even) or V (odd) of block r / 2, in slot r % n_slots
        const uint64_t off = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(id_lane, issued >> 1) * page_stride;
        const char *base = ((issued & 1) ? vbase : kbase) + off;
        const uint32_t lane_off = (issued & 1) ? v_src : k_src;
        const uint32_t dst = lds0 + put * kSlotBytes;
        put = put + 1 == n_slots ? 0 : put + 1;
        ++issued;
#pragma unroll
        for (int q = 0; q < kLoads; ++q) load_to_lds16(base + q * 1024, lane_off, dst + q * 1024);
    };
    request();
    request();

    bf16x8 qf[8];
    {
        const int q_row = a.q_rows ? a.q_rows[req] : req;
        const char *qp = static_cast<const char *>(a.q) + ((size_t)q_row * a.num_q_heads + it.kv_head * G + rowc % G) * (kHeadDim * 2);
#pragma unroll
        for (int i = 0; i < 8; ++i) qf[i] = as_bf16x8(ld16(qp + 2 * (16 * i + 8 * h)));
    }
    int lim = it.n_tokens;
    unsigned long long vis = 0;
    if (a.row_leaf) {  // (all three at once)
        const int leaf = a.row_leaf[req], limit = a.row_limit[req];
        const unsigned long long mask = a.row_mask[req];
        if (leaf == it.node && limit - it.tok_begin < it.n_tokens) {  // (else the whole item lies in front of them, and lim stays its end)
            lim = limit - it.tok_begin;
            vis = mask;
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        u32x4 w = __builtin_bit_cast(u32x4, qf[i]);
        asm volatile("" : "+v"(w));
        qf[i] = as_bf16x8(w);
    }
    asm volatile("" : "+v"(lim), "+v"(vis));
    while (issued < n_slots && issued < n_req) request();

    const int ka_slot = 4 * (n >> 3) + (n & 3), ka_page = (n >> 2) & 1;
    const int ka_swz = ka_page | ((((ka_slot >> 1) ^ (ka_slot >> 2)) & 1) << 1);
    const int ka_base = ka_page * kPageBytes + ka_slot * 64;
    const int va_base = h * kPageBytes + n * 32;
    const int va_swz = ((n >> 2) ^ (n >> 3)) & 1;

    f32x16 o[4];
#pragma unroll
    for (int dm = 0; dm < 4; ++dm) o[dm] = zero16();
    float m_ref = -INFINITY, l_run = 0.f;

    int get = 0;
    auto slot = [&]() -> const char * {
        const char *p = smem + get * kSlotBytes;
        get = get + 1 == n_slots ? 0 : get + 1;
        return p;
    };
    auto arrive = [&](int last) {
        wait_slots_in_flight<kLoads>(issued - 1 - last);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // operand i of a block: K 0-7 unit 0, 8-15 unit 1; V the same (2 dm + e)
    auto rd_k = [&](const char *ks, int i) {
        return *reinterpret_cast<const u32x4 *>(ks + (i >> 3) * 2 * kPageBytes + ka_base + ((i & 7) >> 1) * 1024 + (((2 * (i & 1) + h) ^ ka_swz) << 4));
    };
    auto rd_v = [&](const char *vs, int i) {  // in the order of use: unit, e, dm
        const int e = (i >> 2) & 1, dm = i & 3;
        return *reinterpret_cast<const u32x4 *>(vs + (i >> 3) * 2 * kPageBytes + va_base + dm * 1024 + ((e ^ va_swz) << 4));
    };
    constexpr int R = 8;  // operands on their way from LDS
    auto mask = [&](f32x16 (&s)[2], int j, bool last) {
        const int t0 = j * kBlockTokens;
        if (__builtin_amdgcn_ballot_w64(t0 + 64 > lim)) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int tok0 = t0 + 32 * u + 16 * h;
                const int left = it.n_tokens - tok0;
                // bit i: this row sees token tok0 + i: everything before lim, then the bits of vis, nothing behind them
                const int d0 = tok0 - lim;
                const uint32_t before = (1u << min(max(-d0, 0), 16)) - 1u;
                const uint32_t right = (uint32_t)(vis >> (d0 & 63)), left_shifted = (uint32_t)vis << (-d0 & 31);
                const uint32_t seen = before | (d0 >= 64 || d0 <= -16 ? 0u : d0 >= 0 ? right : left_shifted);
#pragma unroll
                for (int i = 0; i < 16; ++i) s[u][i] = ((seen >> i) & 1u) && (!last || i < left) ? s[u][i] : -INFINITY;
            }
        }
    };
    auto block_max = [&](const f32x16 (&s)[2]) {
        float mx = s[0][0];
#pragma unroll
        for (int i = 1; i < 32; ++i) mx = fmaxf(mx, s[i >> 4][i & 15]);
        return mx;
    };
    float m_top = -INFINITY;  // the row's largest reference so far
    auto refer = [&](float mx, bool anew) {  // mx: the next block's largest score; the reference moves to it, the sums with it
        mx = halves_max(mx) * c;
        float base = m_ref;
        if (anew) {
            m_top = fmaxf(m_top, m_ref);
            base = m_top - 4.0f;
        }
        if (anew || __builtin_amdgcn_ballot_w64(mx > m_ref)) {
            const float m_new = fmaxf(mx, base);
            const float alpha = m_new == -INFINITY ? 1.f : fast_exp2(m_ref - m_new);
            m_ref = m_new;
            l_run *= alpha;
#pragma unroll
            for (int dm = 0; dm < 4; ++dm) o[dm] *= alpha;
        }
    };
    // Phase j: s holds the scores of block j on entry, MORE: those of block j + 1 on exit.
    auto phase = [&](auto more_tag, int j, const f32x16 (&s)[2], f32x16 (&sn)[2]) {
        constexpr bool MORE = decltype(more_tag)::value;
        arrive(MORE ? 2 * j + 2 : 2 * j + 1);
        for (int i = 0; i < 2; ++i)
            if (issued < n_req && issued <= 2 * j + n_slots) request();
        if (!active) return;
        const char *vs = slot(), *ks = vs;
        if constexpr (MORE) ks = slot();
        u32x4 op[R];
        auto operand = [&](int i) { return i < 16 ? rd_k(ks, i) : rd_v(vs, i - 16); };
        constexpr int k0 = MORE ? 0 : 16;
#pragma unroll
        for (int i = k0; i < k0 + R; ++i) op[i % R] = operand(i);
        const float mc = m_ref == -INFINITY ? 0.f : m_ref;
        float sum0 = 0.f, sum1 = 0.f, mx = -INFINITY;
        u32x4 pw[4];
        auto pair = [&](int k) {  // probabilities 2 k and 2 k + 1 of the block
            const float p0 = fast_exp2(__builtin_fmaf(s[k >> 3][2 * (k & 7)], c, -mc));
            const float p1 = fast_exp2(__builtin_fmaf(s[k >> 3][2 * (k & 7) + 1], c, -mc));
            sum0 += p0;
            sum1 += p1;
            uint32_t pk = pack_bf16(p0, p1);
            asm volatile("" : "+v"(pk), "+v"(sum0), "+v"(sum1));
            pw[k >> 2][k & 3] = pk;
        };
        if constexpr (!MORE)
#pragma unroll
            for (int k = 0; k < 10; ++k) pair(k);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
        // 16 slots of the first product with ten pairs of exponentials beside them, 16 of the second with the other six and the
        // maximum of the new scores
#pragma unroll
        for (int i = k0; i < 32; ++i) {
            if (i < 16) {
                sn[(i >> 3) & 1] = mfma32(as_bf16x8(op[i % R]), qf[i & 7], (i & 7) == 0 ? zero16() : sn[(i >> 3) & 1]);
            } else {
                u32x4 w = op[i % R];
                if constexpr (!MORE) {
                    const int left = it.n_tokens - (j * kBlockTokens + 32 * ((i - 16) >> 3) + 16 * h), e = (i >> 2) & 1;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int keep = left - 8 * e - 2 * k;
                        w[k] &= keep >= 2 ? 0xFFFFFFFFu : keep <= 0 ? 0u : 0x0000FFFFu;
                    }
                }
                o[i & 3] = mfma32(as_bf16x8(w), as_bf16x8(pw[((i - 16) >> 2) & 3]), o[i & 3]);
            }
            if (i + R < 32) op[i % R] = operand(i + R);
            if (i < 16) {
#pragma unroll
                for (int k = i * 10 / 16; k < (i + 1) * 10 / 16; ++k) pair(k);
            } else if (i < 24) {
#pragma unroll
                for (int k = 10 + (i - 16) * 6 / 8; k < 10 + (i - 15) * 6 / 8; ++k) pair(k);
            } else if constexpr (MORE) {
#pragma unroll
                for (int k = 2 * (i - 24); k < 2 * (i - 24) + 2; ++k) mx = fmaxf(fmaxf(mx, sn[k >> 3][2 * (k & 7)]), sn[k >> 3][2 * (k & 7) + 1]);
                asm volatile("" : "+v"(mx));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
        l_run += sum0 + sum1;
        if constexpr (MORE) {
            if (__builtin_amdgcn_ballot_w64((j + 1) * kBlockTokens + 64 > lim)) {
                mask(sn, j + 1, j + 2 == n_blk);
                mx = block_max(sn);
            }
            refer(mx, (j + 1) % kAnewBlocks == 0);
        }
    };

    f32x16 sa[2] = {zero16(), zero16()}, sb[2];
    arrive(0);
    if (active) {
        const char *ks = slot();
#pragma unroll
        for (int i = 0; i < 16; ++i) sa[i >> 3] = mfma32(as_bf16x8(rd_k(ks, i)), qf[i & 7], sa[i >> 3]);
        mask(sa, 0, n_blk == 1);
        refer(block_max(sa), false);
    }
    int j = 0;
    for (; j + 2 < n_blk; j += 2) {
        phase(std::true_type{}, j, sa, sb);
        phase(std::true_type{}, j + 1, sb, sa);
    }
    if (j + 1 < n_blk) {
        phase(std::true_type{}, j, sa, sb);
        sa[0] = sb[0];
        sa[1] = sb[1];
        ++j;
    }
    phase(std::false_type{}, j, sa, sb);
    if (!active) return;

    const float L = halves_sum(l_run);
    const float inv = L > 0.f ? 1.0f / L : 0.f;
    float amax = 0.f;
#pragma unroll
    for (int dm = 0; dm < 4; ++dm)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            o[dm][i] *= inv;
            amax = fmaxf(amax, fabsf(o[dm][i]));
        }
    amax = halves_max(amax);
    float up, down;
    part_factors(amax, up, down);
    // (both halves of a row's lanes take part in every exchange)
    uint16_t *op = a.o_parts + ((size_t)(req * a.num_q_heads + it.kv_head * G + rowc % G) * a.max_parts + it.part_slot) * kHeadDim + 8 * h;
#pragma unroll
    for (int dm = 0; dm < 4; ++dm)
#pragma unroll
        for (int q4 = 0; q4 < 4; q4 += 2) {
            u32x2 w[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int i = 4 * (q4 + k);
                w[k] = u32x2{pack_f16(o[dm][i] * up, o[dm][i + 1] * up), pack_f16(o[dm][i + 2] * up, o[dm][i + 3] * up)};
            }
            const u32x4 both = join_halves(w[0], w[1]);
            if (row < rows) *reinterpret_cast<u32x4 *>(op + 32 * dm + 8 * q4) = both;
        }
    if (row < rows && h == 0) {
        const size_t part = (size_t)(req * a.num_q_heads + it.kv_head * G + row % G) * a.max_parts + it.part_slot;
        a.down_parts[part] = down;
        a.lse_parts[part] = partial_lse(m_ref, L);
    }
}

}  // namespace tall

}  // namespace hkv
