// Internal interface between the host side of the library (api.cpp) and its gfx950 kernels.
// Not part of the C ABI.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

namespace hkv {

constexpr int kPage = 16;
constexpr int kHeadDim = 128;
constexpr int kBlockElems = kPage * kHeadDim;  // elements of one (page, head) K or V block

// One decode workgroup: the tokens [tok_begin, tok_begin + n_tokens) of one tree node, one KV
// head, applied to n_req of the requests below the node (n_req * G query rows, at most 64; in bf16 plans with tall tiles 128).
struct DecodeItem {
    int32_t page_off;   // index of the item's first page in the plan's page list
    int32_t n_tokens;   // tokens of this item; only the node's last item may end inside a page
    int32_t kv_head;
    int32_t req_off;    // index of the item's first request in the node->request CSR values
    int32_t n_req;
    int32_t part_slot;  // position of this item among the partials of every row below the node:
                        // row (request r, q head h) writes partial (r*Hq + h)*max_parts + part_slot
    int32_t tok_begin;  // first token within the node (multiple of 16)
    int32_t node;
};

// One prefill workgroup: n_q consecutive new tokens of one request, all G query heads of one KV head.
struct PrefillTile {
    int32_t req;
    int32_t q_begin;    // first new token of the tile within the request's suffix
    int32_t n_q;
    int32_t kv_head;
    int32_t q_row0;     // row of that token in q / out: cu_q[req] + q_begin
    int32_t prefix_len; // cached tokens in front of the request's suffix
    int32_t kv_len;
    int32_t bt_off;     // offset of the request's row in the uploaded block table
};

// A run of a prefill tile's 64-token key blocks, one workgroup's work where tiles are split along their keys.
struct PrefillSegment {
    PrefillTile t;      // the tile, its positions, lengths and table offset moved to the segment's first key
    int32_t kv_end;     // keys of the segment (a multiple of 64 unless it is the tile's last)
    int32_t part;       // partial result it writes; -1: the segment is the whole tile and writes the output itself
};
// A tile cut into segments: its partials are part0 .. part0 + n_parts - 1.
struct PrefillSplitTile {
    PrefillTile t;
    int32_t part0;
    int32_t n_parts;
};
// One partial of a split tile: 256 rows of unnormalised fp32 o in the accumulators' register order, then for each of the eight
// 32-row tiles the softmax references of its rows and their row sums.  (Whether the running-maximum path was taken is kept apart,
// in PrefillLaunch::part_bail.)
constexpr size_t kSplitPartFloats = 256 * kHeadDim + 2 * 256;

struct PoolView {
    const void *k_pages;
    const void *v_pages;
    const float *k_scale;
    const float *v_scale;
    int32_t num_kv_heads;
    int32_t dtype;
};

struct DecodeLaunch {
    PoolView pool;
    const void *q;               // [n_req][Hq][128] bf16
    const DecodeItem *items;     // device
    const int32_t *pages;        // device: the plan's page list
    const int32_t *node_req_idx; // device: node->request CSR values
    uint16_t *o_parts;           // [n_req*Hq*max_parts][128] fp16, each partial times a power of two of its own ...
    float *lse_parts;            // [n_req*Hq*max_parts]
    float *down_parts;           // [n_req*Hq*max_parts]: ... whose reciprocal is kept here
    int32_t n_items;
    int32_t num_q_heads;
    int32_t max_parts;
    float scale;
    // Several query tokens per request (null otherwise): row r of q is query token r % T of request
    // r / T; inside the node row_leaf[r] it sees the first row_limit[r] tokens (everything before the
    // request's T newest tokens) and, of the tokens behind them, number j iff bit j of row_mask[r] is
    // set (a causal run, or the ancestors in a tree of drafted tokens); every other node of its path
    // it sees whole.
    const int32_t *row_leaf;     // device [n_req * T]
    const int32_t *row_limit;    // device [n_req * T]
    const unsigned long long *row_mask;  // device [n_req * T]
    // Items [0, n_single) get a workgroup each; the items behind them (short, at most 16 rows) are run
    // four to a workgroup, one per wavefront.
    int32_t n_single;
    // LDS stages of 16 KiB a workgroup owns (3..5; at least 4 where has_shared): the ring of items shared by more than
    // 16 query rows.  The launch reserves n_stages * 16 KiB of LDS per workgroup.
    int32_t n_stages;
    // fp8 pools: run both products on the fp8 matrix instruction (codes of K and V as they are, query
    // and probabilities as two e4m3 terms each) instead of widening the codes to bf16.
    int32_t fp8_matrix;
    // Row r of the plan reads row q_rows[r] of q (device; null: row r).  Partials stay indexed by r.
    const int32_t *q_rows;
    int32_t has_shared;          // items shared by more than 16 query rows are run by shared::body
    int32_t restart_tokens;      // bf16 pools: after so many tokens such an item takes its rows' references anew (a multiple of 64)
};
// Whole paths instead of items (of the base, what describes items is not read): a record of path_stride ints per leaf and up
// to 16 / G of its rows, run by a workgroup per KV head, which writes out / lse_out (may be null) itself.
struct DecodePathLaunch : DecodeLaunch {
    const int32_t *paths;        // device
    int32_t path_stride;
    int32_t n_paths;
    void *out;
    float *lse_out;
};
// A path's record: {blocks, rows, position of the leaf's first token, 0}, the rows of the plan (16 slots), their rows of q /
// out, then the path's blocks as id | (16 - tokens in the block) << kPathIdBits.
constexpr int kPathRows = 4, kPathQRows = 20, kPathBlocks = 36;
constexpr int kPathIdBits = 27, kPathIdMask = (1 << kPathIdBits) - 1;

struct PrefillLaunch {
    PoolView pool;
    const void *q;
    const PrefillTile *tiles;    // device
    const int32_t *block_table;  // device
    void *out;
    float *lse_out;              // may be null
    int32_t n_tiles;
    int32_t num_q_heads;
    float scale;
    unsigned int *fallback_tiles;  // device, may be null: counts the tiles that had to repeat with a running maximum
    // Tiles split along their keys (n_workers > 0): worker w runs the segments seg_begin[w] .. seg_begin[w + 1] - 1, then a
    // second kernel combines the partials of the n_split cut tiles.
    const PrefillSegment *segments;     // device
    const int32_t *seg_begin;           // device [n_workers + 1]
    const PrefillSplitTile *split;      // device
    float *part_data;                   // device, kSplitPartFloats per partial
    int32_t *part_bail;                 // device, one per partial
    int32_t n_workers;
    int32_t n_split;
};

struct PoolWriteLaunch {
    void *k_pages;
    void *v_pages;
    float *k_scale;
    float *v_scale;
    int32_t num_kv_heads;
    int32_t dtype;
    const int32_t *page_ids;     // device
    int32_t n_pages;
    int32_t first_slot;
    int32_t n_tokens;
    const void *k_src;
    const void *v_src;
    // One token for each of n_pages sequences instead of one run of tokens (null otherwise): workgroup
    // (i, head) stores source row i at slot slots[i] (0..15) of block page_ids[i]; first_slot and
    // n_tokens are not used.
    const int32_t *slots;        // device
    // The block ids on the host (null: page_ids above): up to kMaxInlineWrite of them travel in the kernel's
    // arguments; page_ids is then not read.  bf16 and fp8 pools, runs of tokens only.
    const int32_t *host_ids;
};
constexpr int kMaxInlineWrite = 960;  // with the rest of the arguments below 4 KiB

// One token for each of up to kMaxInlineAppend sequences, ids and slots by value.
constexpr int kMaxInlineAppend = 256;
struct PoolAppendInline {
    PoolWriteLaunch base;        // page_ids / slots / first_slot / n_tokens unused; n_pages = number of tokens
    int32_t block[kMaxInlineAppend];
    uint8_t slot[kMaxInlineAppend];
};

// One decode step's change to an uploaded growing plan, for up to kMaxInlineAppend requests: the items
// listed in grow_items get one token more, and request r's new 16-token block (if it opens one) is
// entered at position block_pos[r] of the plan's block list.
struct PlanGrowInline {
    DecodeItem *items;           // device
    int32_t *pages;              // device
    const int32_t *grow_items;   // device, n_grow entries
    int32_t n_grow;
    int32_t n_req;
    int32_t new_block[kMaxInlineAppend];  // -1: none
    int32_t block_pos[kMaxInlineAppend];
};

// Whole-page copies inside one pool (copy-on-write of pages that several holders share).
constexpr int kMaxCopyPairs = 32;
struct PoolCopyLaunch {
    PoolView pool;
    int32_t blocks_per_page;     // a page is this many consecutive 16-token blocks
    int32_t n;
    int32_t src[kMaxCopyPairs];
    int32_t dst[kMaxCopyPairs];
};

// fp8 pages -> bf16 pages of a scratch pool (page i of the scratch = src_pages[i] of the pool), so that
// the matrix-core prefill kernel can read an fp8 pool.
struct PoolDequantLaunch {
    PoolView pool;               // the fp8 pool
    const int32_t *src_pages;    // device [n_pages]
    int32_t n_pages;
    void *k_dst;                 // device, n_pages * num_kv_heads * 2048 bf16, bf16 block format
    void *v_dst;
};

// fp32 pools: a workgroup per (query token, KV head, pair of its query heads), no sharing between requests (rows_fp32.hip).
struct RowsLaunch {
    PoolView pool;
    const float *q;              // [n_q_tokens][Hq][128] fp32
    const int32_t *block_table;  // device [n_rows_of_table][max_pages]
    const int32_t *row_req;      // device [n_q_tokens]: row of the block table
    const int32_t *row_len;      // device [n_q_tokens]: keys the token sees
    float *out;                  // [n_q_tokens][Hq][128] fp32
    float *lse_out;              // may be null
    int32_t n_q_tokens;
    int32_t num_q_heads;
    int32_t max_pages;
    float scale;
    // Few rows: their keys cut into n_parts shares, a workgroup each, whose results part_data (device, kRowPartFloats per row of out and
    // share) holds for a second kernel; n_parts <= 1: whole rows.
    int32_t n_parts;
    float *part_data;
};
constexpr int kMaxRowParts = 32;
constexpr int kRowPartFloats = kHeadDim + 4;  // o, reference, row sum; 16-byte pieces
constexpr int kRowWorkgroups = 256;           // what fills the chip: rows are cut, or given fewer of their heads a workgroup, until there are so many
// Shares that the keys of a decode plan's rows are cut into (1: rows stay whole), where the caller gives room for their results.  Few rows
// leave compute units idle, and a row's workgroup takes in no more than one can: shares of up to four heads, down to 128 keys each, until
// every compute unit has one.  They save their part of the walk, 0.13 us a page, less 4.5 us for the second kernel and a second start, so
// shorter rows stay whole: over 518 keys 9.6 -> 10.6 us for one request (32 / 8 heads), 11.2 -> 12.9 for 16; over 1020 keys 14.3 -> 10.6 for 2.
// But keys that are read all at once come slower than a walk reads them: 0.1 us more for each MB beyond 40 (ratio 1: 0.13 beyond 15) of the
// plan's K/V.  Not so where it comes from memory anyway (128 MB and more, three shares and more), where the walk is long (100 pages; ratio 1, three
// shares and more, 160), and where a row's keys are read from memory twice without shares, by workgroups of two heads on different XCDs.  1214
// plans of 64 to 400 pages, ratios 1 to 16, keys shared in all proportions, time over the whole rows', K/V from the last-level cache
// and from memory: where shares are taken 0.21 to 1.14 and 0.33 to 0.98 (0.78 and 0.71 in the mean), else 0.84 to 1.53 (16 requests x 4 / 4
// heads over 1021 keys of their own 15.5 -> 23.8 us) and 0.68 to 1.13 (1.10 and 0.90).
inline int row_shares(int64_t n_rows, int num_kv_heads, int group, int max_pages, double plan_mb) {
    const int heads = group <= 2 ? group : 4;
    const int64_t units = n_rows * num_kv_heads * ((group + heads - 1) / heads);
    int64_t shares = units > 0 ? kRowWorkgroups / units : 1;
    if (shares > max_pages / 8) shares = max_pages / 8;
    if (shares > kMaxRowParts) shares = kMaxRowParts;
    if (shares < 2 || max_pages < (shares == 2 ? 72 : 64)) return 1;
    if (group > 2 && num_kv_heads % 8 != 0) return (int)shares;
    const double saved = 0.13 * max_pages * (1.0 - 1.0 / (double)shares) - 4.5;
    const bool far = plan_mb >= 128.0 && shares > 2, long_rows = group == 1 ? max_pages >= 160 && shares > 2 : max_pages >= 100;
    return far || long_rows || plan_mb <= (group == 1 ? 15.0 + saved / 0.13 : 40.0 + saved / 0.1) ? (int)shares : 1;
}
// Query heads of a KV head that a workgroup of theirs takes: they share its K/V reads, which are what long rows are bound by (a compute unit
// takes in about 110 bytes per ns).  Four, where every compute unit then still has a workgroup, for half as many workgroups that cost 1.25 times
// as much each: what counts is how many rounds of them a compute unit gets.  1277 shapes, head ratios 3 to 16, keys shared or private, time
// over that with two heads:
// - rows of more than 16 pages: 0.51 to 0.96 with fewer rounds (32 requests x 32 / 8 heads over 1024 + 256 tokens 36.0 -> 25.0 us, 16 x 64 / 8
//   32.8 -> 21.4), 1.04 to 1.17 with as many (17 to 21 requests x 40 / 8, two rounds either way);
// - 9 to 16 pages: 0.56 to 0.97 with up to 0.7 of the rounds (1.05 at worst, private keys of 33 requests x 32 / 8), 0.94 to 1.19 above;
// - 5 to 8 pages: 0.61 to 1.02 with up to 0.6 of five rounds and more, of fewer 0.96 to 1.22 (33 x 32 / 8 over 48 + 30 7.9 -> 8.7).  Where the
//   workgroups of a row's KV head lie on different XCDs (neighbours in the grid are num_kv_heads apart) two heads read private keys from
//   memory twice: 0.61 to 0.85, shared ones up to 1.13;
// - ratios that four does not divide, 5 to 8 pages: 33 x 40 / 8 over 96 + 17 10.4 -> 11.1; up to 4 pages 48 x 32 / 8 over 16 + 30 7.7 -> 8.6.
inline int row_heads_per_workgroup(int64_t n_rows, int num_kv_heads, int group, int max_pages, bool in_shares) {
    if (group <= 2) return group;
    if (in_shares) return 4;
    const int64_t n4 = n_rows * num_kv_heads * ((group + 3) / 4), n2 = n_rows * num_kv_heads * ((group + 1) / 2);
    const int64_t four = (n4 + kRowWorkgroups - 1) / kRowWorkgroups, two = (n2 + kRowWorkgroups - 1) / kRowWorkgroups;
    if (n4 < kRowWorkgroups || max_pages <= 4) return 2;
    if (max_pages > 16) return four < two ? 4 : 2;
    if (max_pages > 8) return 10 * four <= 7 * two ? 4 : 2;
    if (group % 4 != 0) return 2;
    return num_kv_heads % 8 != 0 ? (10 * four <= 7 * two ? 4 : 2) : two >= 5 && 10 * four <= 6 * two ? 4 : 2;
}

// Largest token count of a decode item that is shared by more than 16 query rows.
constexpr int kMaxSharedItemTokens = 2048;

// Decode items shared by more than kMinTileItemRows query rows are run by the 256-row tile kernel (the
// prefill kernel in its second role), on a stream of its own next to the kernel that streams the rest.
constexpr int kMinTileItemRows = 65;
constexpr int kMaxTileItemTokens = 8192;  // tokens per such item
constexpr int kScaleSlots = 512;          // pages whose fp8 scales the tile kernel keeps in LDS
struct DecodeTilesLaunch {
    PoolView pool;
    const void *q;               // [n_req][Hq][128] bf16
    const DecodeItem *items;     // device: the items of this kernel (at most 256 / G requests each)
    const int32_t *pages;        // device: the plan's block list
    const int32_t *node_req_idx; // device: node->request CSR values
    uint16_t *o_parts;           // as DecodeLaunch::o_parts
    float *lse_parts;
    float *down_parts;
    int32_t n_items;
    int32_t num_q_heads;
    int32_t max_parts;
    float scale;
    int32_t n_workgroups;        // persistent workgroups: workgroup w runs items w, w + n_workgroups, ...
    const int32_t *q_rows;       // device, may be null: as DecodeLaunch::q_rows
};

// A prefill tile of up to 64 rows runs as token halves (tile_body.h) where it has more keys than this: below, bringing the halves together
// costs what they save (16 x 12 new tokens over 2048, 32 / 8 heads, 33.4 -> 25.4 us, 30 x 16 over 512 14.3 -> 12.5, over 256 10.9 ->
// 10.3; over 128 9.3 either way, 32 x 16 over 64 8.6 -> 8.8).
constexpr int kPrefillHalvesTokens = 256;
// Query tokens per prefill workgroup for a given group size G (rows per workgroup / G).
int prefill_tile_tokens(int group);
// Both kinds of decode items in one launch (no item of `a` may be shared by more than 16 query rows).
hipError_t launch_decode_fused(const DecodeLaunch &a, const DecodeTilesLaunch &d, hipStream_t s,
                               hipEvent_t ev_begin = nullptr, hipEvent_t ev_end = nullptr);

hipError_t launch_pool_write(const PoolWriteLaunch &a, hipStream_t s);
// src may be pinned host memory (its device-side address); bytes is rounded down to a multiple of 16
hipError_t launch_upload(const void *src, void *dst, size_t bytes, hipStream_t s);
hipError_t launch_pool_append_inline(const PoolAppendInline &a, hipStream_t s);
// both in one launch: workgroup (r, head) stores request r's token and lengthens the leaf's item of that head
hipError_t launch_decode_step_append(const PoolAppendInline &w, const PlanGrowInline &g, hipStream_t s);
hipError_t launch_plan_grow_inline(const PlanGrowInline &a, hipStream_t s);
hipError_t launch_pool_copy(const PoolCopyLaunch &a, hipStream_t s);
hipError_t launch_pool_dequant(const PoolDequantLaunch &a, hipStream_t s);
// Once per device (later calls only read the result), with that device current and outside graph capture:
// allows the decode kernels their LDS and looks up the device's static workspace (kStaticWorkspaceBytes
// bytes, 256-byte aligned), returned through static_ws unless that is null.  Safe from several threads.
constexpr size_t kStaticWorkspaceBytes = (size_t)32 << 20;
hipError_t prepare_decode_device(void **static_ws);
hipError_t launch_decode(const DecodeLaunch &a, hipStream_t s, hipEvent_t ev_begin = nullptr, hipEvent_t ev_end = nullptr);
// waves: 4 or 8 wavefronts per workgroup
hipError_t launch_decode_paths(const DecodePathLaunch &a, int waves, hipStream_t s, hipEvent_t ev_begin = nullptr, hipEvent_t ev_end = nullptr);
hipError_t launch_rows_fp32(const RowsLaunch &a, hipStream_t s);
hipError_t launch_pool_write_fp32(const PoolWriteLaunch &a, hipStream_t s);
hipError_t launch_prefill(const PrefillLaunch &a, hipStream_t s);
hipError_t launch_decode_tiles(const DecodeTilesLaunch &a, hipStream_t s, hipEvent_t ev_begin = nullptr, hipEvent_t ev_end = nullptr);
hipError_t launch_lse_merge(const float *o_parts, const float *lse_parts, const int32_t *row_indptr,
                            const int32_t *part_idx, int32_t n_rows, void *out, int32_t out_dtype,
                            float *lse_out, hipStream_t s);
// out_rows (device, may be null): the rows of group g = row / rows_per_count are written to group out_rows[g]
// of out / lse_out instead of group g.
// down_parts (device, may be null): o_parts holds fp16 values, partial n to be multiplied by down_parts[n] (the
// decode plans' own partials), instead of floats.
hipError_t launch_lse_merge_dense(const void *o_parts, const float *lse_parts, const int32_t *part_count,
                                  int32_t rows_per_count, int32_t max_parts, int32_t n_rows, void *out,
                                  int32_t out_dtype, float *lse_out, hipStream_t s, hipEvent_t ev_begin = nullptr,
                                  hipEvent_t ev_end = nullptr, const int32_t *out_rows = nullptr,
                                  const float *down_parts = nullptr);

}  // namespace hkv
