// Decode items shared by 17 to 64 query rows (device code, called by rows_body.h): one workgroup of four wavefronts
// applies a chunk of a prefix-tree node to up to two 32-row tiles.  (Shared prefix KV computed once and reused by
// every call below it: Section 5, "Proactive Cache Management".)
//
// Matrix-core mapping (v_mfma_f32_32x32x16_bf16, wavefront = row tile rt x token half th of a 64-token block):
//   S^T = K * Q^T   A = 32 tokens x 16 dims of K, B = 16 dims x 32 query rows, D[token][row]
//   O^T = V^T * P^T A = 32 dims x 16 tokens of V^T, B = 16 tokens x 32 query rows, D[dim][row]
// The M index of the score tile is permuted so that the lower half of the wavefront holds the 16 tokens of the
// unit's first page and the upper half those of its second: a lane's 16 scores are the 16 slots of one page in
// order, which is a ready B operand for the second product, one fp8 scale per lane, and 16-byte reads of V.
//
// What bounds it.  HBM hands a compute unit about 9 bytes per cycle, i.e. a 16 KiB block of K and V every 1800
// cycles; the vector instructions of a block (and, for fp8 pools, the widening of its codes to bf16) have to stay
// below that.  With a 16-row tile per wavefront over all tokens they did not: every wavefront read every K/V operand
// from LDS and widened it for 16 rows only, about 24 vector instructions per score and lane.  Here an operand
// serves 32 rows and each wavefront touches half of the tokens.  bf16 pools: the reference is the running maximum.  The
// probabilities are rounded to bf16, whose relative error is smallest just below a power of two (and nil at it): with the
// maximum as reference that is where a row's heaviest weights lie, with any other they fall anywhere in the binade and the
// error of a result grows by 6 % (0.00219 -> 0.00232 with references up to 8 powers of two behind, 0.00216 this way).
// fp8 pools: a probability is multiplied by its block's V scale before it is rounded, so there is no such place; the
// reference moves only when a score passes it by 8 powers of two, and the accumulators are rescaled once or twice per item.
//
// Latency, not issue rate, is what the first form of this loop ran into (3900 cycles per block with a fifth of them
// busy): an LDS read takes about 200 cycles, so a phase reads its operands in bulk, runs S(j+1) = K(j+1) Q^T beside
// P(j) = exp2(S(j)), then O += V(j) P(j): one barrier per 64-token block.  Measured: 64 rows, 0.8 (fp8) to 0.9 us per block
// alone, 1.1 us for two workgroups of a compute unit from L2 (60 B/ns), 2.9 us bf16 / 1.5 us fp8 from HBM (5.8 / 5.4 TB/s).
// Kernel over 100 requests x 5 heads below ten 8192-token contexts, fp8: 61 -> 47 us; step of 512 rows below 4096 tokens and 64
// below each of 8 x 1024, bf16: 39.7 -> 36.0 us.
// K and V travel through one LDS ring of half-blocks in the order K(0), V(0), K(1), V(1), ...
#pragma once
#include "hkv_device.h"

namespace hkv {

namespace shared {

constexpr int kWaves = 4;
constexpr int kBlockTokens = 64;   // one half-step: K or V of four pages

// Waits until at most n vector-memory operations of this wavefront are outstanding (and every LDS read has
// returned, so that the slot it read may be overwritten behind the barrier that follows).
template <int N>
__device__ __forceinline__ void wait_loads() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"i"(N) : "memory");
}
// The same for a number of ring slots, PER_SLOT operations each (wavefront-uniform, 0 .. 7).
template <int PER_SLOT>
__device__ __forceinline__ void wait_slots_in_flight(int slots) {
    switch (slots) {
        case 0: wait_loads<0>(); break;
        case 1: wait_loads<PER_SLOT>(); break;
        case 2: wait_loads<2 * PER_SLOT>(); break;
        case 3: wait_loads<3 * PER_SLOT>(); break;
        case 4: wait_loads<4 * PER_SLOT>(); break;
        case 5: wait_loads<5 * PER_SLOT>(); break;
        case 6: wait_loads<6 * PER_SLOT>(); break;
        default: wait_loads<7 * PER_SLOT>(); break;
    }
}

__device__ __forceinline__ float halves_max(float v) {  // over lanes l and l ^ 32
    const uint32_t x = __float_as_uint(v);
    const auto b = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float halves_sum(float v) {
    const uint32_t x = __float_as_uint(v);
    const auto b = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// FP8: the pool holds e4m3 codes with a scale per 16-token block and head.  smem: a.n_stages * 16 KiB.
template <bool FP8>
__device__ __forceinline__ void body(const DecodeLaunch &a, const DecodeItem &it, char *smem, const int wave, const int lane) {
    constexpr int kPageBytes = kBlockElems * (FP8 ? 1 : 2);
    constexpr int kSlotBytes = 4 * kPageBytes;
    constexpr float kLazy = FP8 ? 8.0f : 0.0f;      // a reference moves when a score passes it by this many powers of two
    constexpr int kLoads = kPageBytes / 1024;       // LDS-direct loads per wavefront and half-step (wavefront w: page w)
    constexpr int kKReads = FP8 ? 4 : 8;            // 16-byte K operand reads per 32-token unit and lane
    const int Hkv = a.pool.num_kv_heads, G = a.num_q_heads / Hkv;
    const int rows = it.n_req * G;
    const int n = lane & 31, h = lane >> 5;
    const int rt = wave & 1, th = wave >> 1;
    const bool active = 32 * rt < rows;             // wavefront-uniform
    const float c = a.scale * kLog2e;
    const int n_blk = (it.n_tokens + kBlockTokens - 1) / kBlockTokens;
    const int last_page = (it.n_tokens - 1) >> 4;
    const uint32_t page_stride = (uint32_t)Hkv * kPageBytes;
    const char *kbase = static_cast<const char *>(a.pool.k_pages) + (size_t)it.kv_head * kPageBytes;
    const char *vbase = static_cast<const char *>(a.pool.v_pages) + (size_t)it.kv_head * kPageBytes;

    // Lane b holds the id of page 4 b + wave of the item: the page this wavefront fetches in block b (the planner
    // keeps these items at 2048 tokens = 32 blocks or fewer).  Pages past the end are clamped: in bounds, masked below.
    const int32_t *ids = a.pages + it.page_off;
    const int id_lane = ids[min(4 * lane + wave, last_page)];
    // In the same round trip as the ids (the requests below wait for those, and what stands behind them is loaded one trip later), as
    // the three words of a row's visibility are: with these and the partials going out in pieces of 16 bytes instead of 8, 512 rows
    // below 4096 tokens and 64 below each of 8 x 1024 35.13 -> 34.55 us (100 requests x 5 heads over fp8 53.31 -> 52.76, no more than runs differ).
    const int row = 32 * rt + n, rowc = min(row, rows - 1);
    const int req = a.node_req_idx[it.req_off + rowc / G];
    // fp8: lane 32 j + b holds the scales of page 4 b + 2 th + j, the page whose tokens half j of the wavefront scores
    float ksc_lane = 1.f, vsc_lane = 1.f;
    if constexpr (FP8) {
        const size_t id = (size_t)ids[min(4 * n + 2 * th + h, last_page)] * Hkv + it.kv_head;
        ksc_lane = a.pool.k_scale[id];
        vsc_lane = a.pool.v_scale[id];
    }
    auto of_block = [&](float v, int b) {  // this lane half's value for block b
        const float lo = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), b));
        const float hi = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), b + 32));
        return h ? hi : lo;
    };

    // LDS image of a slot: four pages; a K page as [1 KiB chunk][slot][4 units of 16 B], unit ^= f(page, slot); a V page
    // as [dim][2 units of 8 tokens], unit ^= g(dim) (bf16) resp. [dim][16 codes] (fp8).  f and g spread the 16-byte
    // pieces that neighbouring lanes read over the banks, for 128- and for 256-byte accesses per cycle.
    const int l_slot = lane >> 2;
    const uint32_t k_src = (uint32_t)(l_slot * 64 + (((lane & 3) ^ ((wave & 1) | ((((l_slot >> 1) ^ (l_slot >> 2)) & 1) << 1))) << 4));
    const uint32_t v_src = FP8 ? (uint32_t)lane * 16 : (uint32_t)((lane >> 1) * 32 + (((lane & 1) ^ (((lane >> 3) ^ (lane >> 4)) & 1)) << 4));
    const int n_slots = min(a.n_stages * (16384 / kSlotBytes), 9);  // 4 .. 9 (the launch gives at least 4 stages)
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

    // The first block is requested in front of the queries, the rest of the ring behind them: what the compiler loads
    // itself has to be waited for before the loop (it would otherwise wait inside it, for everything in flight), and
    // that wait should find as little as possible in front of it.
    request();
    request();

    // Q^T operands of this lane's row; rows past the item's end repeat its last row (their results are not stored)
    bf16x8 qf[8];
    {
        const int q_row = a.q_rows ? a.q_rows[req] : req;
        const char *qp = static_cast<const char *>(a.q) + ((size_t)q_row * a.num_q_heads + it.kv_head * G + rowc % G) * (kHeadDim * 2);
        // bf16: k-step i covers dims 16 i + 8 h ..; fp8: k-steps 2 i, 2 i + 1 the two halves of dims 32 i + 16 h ..
#pragma unroll
        for (int i = 0; i < 8; ++i) qf[i] = as_bf16x8(ld16(qp + 2 * (FP8 ? 32 * (i >> 1) + 16 * h + 8 * (i & 1) : 16 * i + 8 * h)));
    }
    // Tokens of this item that the row may see: all, unless this is the node that holds its request's newest tokens
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
    asm volatile("" : "+v"(lim), "+v"(vis), "+v"(ksc_lane), "+v"(vsc_lane));
    while (issued < n_slots && issued < n_req) request();

    // this lane's operand positions in a slot
    const int ka_slot = 4 * (n >> 3) + (n & 3), ka_page = (n >> 2) & 1;
    const int ka_swz = ka_page | ((((ka_slot >> 1) ^ (ka_slot >> 2)) & 1) << 1);
    const int ka_base = (2 * th + ka_page) * kPageBytes + ka_slot * 64;
    const int va_base = (2 * th + h) * kPageBytes + n * (FP8 ? 16 : 32);
    const int va_swz = ((n >> 2) ^ (n >> 3)) & 1;

    f32x16 o[4];  // O^T: dim 32 dm + 8 (i / 4) + 4 h + i % 4 of row n
#pragma unroll
    for (int dm = 0; dm < 4; ++dm) o[dm] = zero16();
    float m_ref = -INFINITY, l_run = 0.f;  // the row's reference (times scale * log2 e); this lane's share of the row sum

    int get = 0;  // slot of the next half-block to be read
    auto slot = [&]() -> const char * {
        const char *p = smem + get * kSlotBytes;
        get = get + 1 == n_slots ? 0 : get + 1;
        return p;
    };
    // Half-blocks up to number `last` have landed for everyone, and everyone is done with the half-blocks of the phase
    // before: their slots take the next requests.
    auto arrive = [&](int last) {
        wait_slots_in_flight<kLoads>(issued - 1 - last);  // (loads complete in order)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    struct KOperands {
        u32x4 w[kKReads];
    };
    auto read_k = [&](KOperands &k, const char *ks) {
#pragma unroll
        for (int i = 0; i < kKReads; ++i) k.w[i] = *reinterpret_cast<const u32x4 *>(ks + ka_base + (i >> 1) * 1024 + (((2 * (i & 1) + h) ^ ka_swz) << 4));
    };
    auto scores = [&](const KOperands &k) {
        f32x16 s = zero16();
#pragma unroll
        for (int i = 0; i < kKReads; ++i) {
            if constexpr (FP8) {
                s = mfma32(fp8x8_to_bf16x8(k.w[i][0], k.w[i][1]), qf[2 * i], s);
                s = mfma32(fp8x8_to_bf16x8(k.w[i][2], k.w[i][3]), qf[2 * i + 1], s);
            } else {
                s = mfma32(as_bf16x8(k.w[i]), qf[i], s);
            }
        }
        return s;
    };
    // Phase j: s holds the scores of block j on entry; MORE: sn those of block j + 1 on exit.  LAST block: may reach past
    // the item's end (garbage slots may hold NaN).
    auto phase = [&](auto more_tag, int j, f32x16 &s, f32x16 &sn) {
        constexpr bool MORE = decltype(more_tag)::value;
        arrive(MORE ? 2 * j + 2 : 2 * j + 1);
        for (int i = 0; i < 2; ++i)
            if (issued < n_req && issued <= 2 * j + n_slots) request();
        if (!active) return;  // no row in this wavefront's tile: it only fetches
        const char *vs = slot();
        KOperands k;
        if constexpr (MORE) read_k(k, slot());

        const int tok0 = j * kBlockTokens + 32 * th + 16 * h;  // token of this lane's score 0
        const int left = it.n_tokens - tok0;                   // valid slots of this lane's page (LAST: possibly below 16)
        if (__builtin_amdgcn_ballot_w64(tok0 + 16 > lim)) {
            // bit i: this row sees token tok0 + i: everything before lim, then the bits of vis, nothing behind them
            const int d0 = tok0 - lim;
            const uint32_t before = d0 >= 0 ? 0u : d0 <= -16 ? 0xFFFFu : (1u << -d0) - 1u;
            const uint32_t drafted = d0 >= 64 ? 0u : d0 >= 0 ? (uint32_t)(vis >> d0) : d0 <= -16 ? 0u : (uint32_t)vis << -d0;
            const uint32_t seen = before | drafted;
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = ((seen >> i) & 1u) && (MORE || i < left) ? s[i] : -INFINITY;
        }
        const float ck = FP8 ? c * of_block(ksc_lane, j) : c;
        float mx = s[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
        mx = halves_max(mx * ck);
        if (__builtin_amdgcn_ballot_w64(mx > m_ref + kLazy)) {
            const float m_new = mx > m_ref + kLazy ? mx : m_ref;
            const float alpha = m_new == -INFINITY ? 1.f : fast_exp2(m_ref - m_new);
            m_ref = m_new;
            l_run *= alpha;
#pragma unroll
            for (int dm = 0; dm < 4; ++dm) o[dm] *= alpha;
        }
        const float mc = m_ref == -INFINITY ? 0.f : m_ref;  // a row that has seen nothing: exp2(-inf) = 0 either way
        const float vsc = FP8 ? of_block(vsc_lane, j) : 1.f;
        if constexpr (MORE) sn = scores(k);
        // (behind the K operands: both at once would not fit beside the accumulators)
        if constexpr (!FP8) __builtin_amdgcn_sched_barrier(0);
        u32x4 vw[FP8 ? 4 : 8];  // V operands: fp8 [dm], bf16 [2 dm + e]
#pragma unroll
        for (int i = 0; i < (FP8 ? 4 : 8); ++i)
            vw[i] = *reinterpret_cast<const u32x4 *>(vs + va_base + (FP8 ? i * 512 : (i >> 1) * 1024 + (((i & 1) ^ va_swz) << 4)));
        float sum0 = 0.f, sum1 = 0.f;
        u32x4 pw[2];  // probabilities, packed
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            const float p0 = fast_exp2(__builtin_fmaf(s[i], ck, -mc)), p1 = fast_exp2(__builtin_fmaf(s[i + 1], ck, -mc));
            sum0 += p0;
            sum1 += p1;
            pw[i >> 3][(i >> 1) & 3] = FP8 ? pack_bf16(p0 * vsc, p1 * vsc) : pack_bf16(p0, p1);
        }
        l_run += sum0 + sum1;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int dm = 0; dm < 4; ++dm) {
                if constexpr (FP8) {
                    uint32_t w0 = vw[dm][2 * e], w1 = vw[dm][2 * e + 1];
                    if constexpr (!MORE) {
                        const int keep = left - 8 * e;
                        w0 &= keep >= 4 ? 0xFFFFFFFFu : keep <= 0 ? 0u : ((1u << (8 * keep)) - 1u);
                        w1 &= keep >= 8 ? 0xFFFFFFFFu : keep <= 4 ? 0u : ((1u << (8 * (keep - 4))) - 1u);
                    }
                    o[dm] = mfma32(fp8x8_to_bf16x8(w0, w1), as_bf16x8(pw[e]), o[dm]);
                } else {
                    u32x4 w = vw[2 * dm + e];
                    if constexpr (!MORE) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int keep = left - 8 * e - 2 * i;
                            w[i] &= keep >= 2 ? 0xFFFFFFFFu : keep <= 0 ? 0u : 0x0000FFFFu;
                        }
                    }
                    o[dm] = mfma32(as_bf16x8(w), as_bf16x8(pw[e]), o[dm]);
                }
            }
    };

    f32x16 sa = zero16(), sb;
    arrive(0);
    if (active) {
        KOperands k;
        read_k(k, slot());
        sa = scores(k);
    }
    // bf16 pools, items longer than the default length: there the reference begins anew, 2^4 below the largest so far, as in
    // rows::body (2048 tokens, error against 64 bits: chunks of 512 0.00215, whole 0.00220, whole with restarts 0.00215).
    float m_top = -INFINITY;
    int restart_at = FP8 ? -1 : a.restart_tokens / kBlockTokens;
    auto restart = [&](int j) {
        if (j != restart_at) return;
        restart_at += a.restart_tokens / kBlockTokens;
        m_top = fmaxf(m_top, m_ref);
        if (m_top == -INFINITY) return;
        const float m_new = m_top - 4.0f, alpha = fast_exp2(m_ref - m_new);
        m_ref = m_new;
        l_run *= alpha;
#pragma unroll
        for (int dm = 0; dm < 4; ++dm) o[dm] *= alpha;
    };
    for (int j = 0; j + 1 < n_blk; ++j) {
        restart(j);
        phase(std::true_type{}, j, sa, sb);
        sa = sb;
    }
    restart(n_blk - 1);
    phase(std::false_type{}, n_blk - 1, sa, sb);

    // The two token halves of a row tile: the upper one hands its results to the lower one through LDS, lane by lane.
    float l_row = halves_sum(l_run);
    f32x4 *xo = reinterpret_cast<f32x4 *>(smem) + rt * (16 * 64) + lane;
    float *xm = reinterpret_cast<float *>(smem + 2 * 16 * 64 * sizeof(f32x4)) + rt * 128 + lane;
    static_assert(2 * 16 * 64 * sizeof(f32x4) + 2 * 128 * sizeof(float) <= 3 * 16384, "hand-over buffer inside the smallest ring");
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();  // the ring has been read
    if (active && th == 1) {
#pragma unroll
        for (int k = 0; k < 16; ++k) xo[64 * k] = f32x4{o[k >> 2][4 * (k & 3)], o[k >> 2][4 * (k & 3) + 1], o[k >> 2][4 * (k & 3) + 2], o[k >> 2][4 * (k & 3) + 3]};
        xm[0] = m_ref;
        xm[64] = l_row;
    }
    __syncthreads();
    if (!active || th == 1) return;
    const float m1 = xm[0], l1 = xm[64];
    const float M = fmaxf(m_ref, m1), Mc = M == -INFINITY ? 0.f : M;
    const float w0 = fast_exp2(m_ref - Mc), w1 = fast_exp2(m1 - Mc);
    const float L = l_row * w0 + l1 * w1;
    const float inv = L > 0.f ? 1.0f / L : 0.f;  // a row that saw no token of this item delivers the empty partial (o = 0, lse = -inf)
    float amax = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const f32x4 x = xo[64 * k];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float &v = reinterpret_cast<float *>(&o[k >> 2])[4 * (k & 3) + j];
            v = (v * w0 + x[j] * w1) * inv;
            amax = fmaxf(amax, fabsf(v));
        }
        __builtin_amdgcn_sched_barrier(0);
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
        a.lse_parts[part] = partial_lse(M, L);
    }
}

}  // namespace shared

}  // namespace hkv
