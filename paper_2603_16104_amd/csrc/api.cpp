// Host side of the heliumkv C ABI: pool bookkeeping, forest validation and flattening, work
// planning, argument checks, kernel launches.  All arithmetic on K/V/Q lives in the kernels.
#include "../../include/heliumkv.h"
#include "hkv_internal.h"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <new>
#include <numeric>
#include <string>
#include <unordered_map>
#include <vector>

using namespace hkv;

// ---------------------------------------------------------------------------------------------
// errors
namespace {
thread_local std::string g_err;
}

namespace hkv {
// records the thread-local message and returns the code (shared with the other host files)
int fail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}
}  // namespace hkv

namespace {

int fail_hip(hipError_t e, const char *what) {
    return fail(HKV_EHIP, "%s: %s", what, hipGetErrorString(e));
}

#define HKV_HIP(call)                                  \
    do {                                               \
        hipError_t e_ = (call);                        \
        if (e_ != hipSuccess) return fail_hip(e_, #call); \
    } while (0)

size_t elem_bytes(int dtype) { return dtype == HKV_BF16 ? 2 : dtype == HKV_FP8_E4M3 ? 1 : 4; }

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// What the planner needs to know of the chip: compute units, and how many workgroups of the per-node decode
// kernel one of them holds (three with bf16 pools, two with fp8 pools: registers).  Asked of the current device;
// plans built without a device (HKV_PLAN_HOST_ONLY on a machine without a GPU) assume an MI355X.
struct ChipShape {
    int n_cu = 256;
    int lds_per_cu = 160 * 1024;
};
ChipShape chip_shape() {
    ChipShape c;
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) {
        if (prop.multiProcessorCount > 0) c.n_cu = prop.multiProcessorCount;
        if (prop.maxSharedMemoryPerMultiProcessor > 0) c.lds_per_cu = (int)prop.maxSharedMemoryPerMultiProcessor;
    } else {
        (void)hipGetLastError();  // no device: not an error of the caller's
    }
    return c;
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// opaque objects
struct hkv_decode_plan {
    hkv_pool *pool = nullptr;
    int32_t n_req = 0, num_q_heads = 0, group = 0, n_parts = 0, max_parts = 1;
    std::vector<hkv_node> key_nodes;        // the caller's forest: key of the one-shot cache
    std::vector<int32_t> key_pages, req_leaf;
    std::vector<hkv_node> nodes;            // the same forest in 16-token blocks (page_begin, n_pages into node_pages)
    std::vector<int32_t> node_pages;
    std::vector<DecodeItem> items;
    // Items shared by kMinTileItemRows query rows or more (up to 256 / G requests each): run by the 256-row
    // tile kernel on tile_workgroups persistent workgroups, on a stream of the plan's own next to the kernel
    // that runs `items` (or in front of it on the caller's stream when concurrent is false).
    std::vector<DecodeItem> tile_items;
    int32_t tile_workgroups = 0;
    // Small steps: whole paths instead of items, one launch (path_waves wavefronts per workgroup; 0: items)
    std::vector<int32_t> paths;
    int32_t path_stride = 0, n_paths = 0, path_waves = 0;
    double paths_us = 0, items_us = 0;  // estimates of a step; paths_us = 0: paths are out of the question, items_us is not asked for
    int32_t *d_paths = nullptr;
    int32_t restart_tokens = kMaxSharedItemTokens;  // a stretch of a shared node's item with one reference per row
    bool row_visibility = false;  // several query tokens per request: rows see their last node in part
    bool concurrent = true;
    bool fused = false;  // both kinds of items go out as one launch (no item of `items` has more than 16 rows)
    hipStream_t side = nullptr;
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    hipEvent_t ev_tile[2] = {nullptr, nullptr};  // profiling: begin/end of the tile kernel
    std::vector<int32_t> node_req_indptr, node_req_idx, part_count;
    // one device allocation holding items | pages | node_req_idx | part_count | tile_items
    void *dev = nullptr;
    DecodeItem *d_items = nullptr, *d_tile_items = nullptr;
    int32_t n_single = 0;  // items [0, n_single) run one per workgroup, the rest four per workgroup
    int32_t n_stages = 3;  // LDS stages of 16 KiB per workgroup of the per-node kernel
    bool has_shared = false;  // items of `items` shared by more than 16 query rows are run by shared::body
    int tile_form = 0;  // bf16 pools: -1 never, 1 always shared::body, 2 with tall tiles (HKV_PLAN_NARROW_TILES, _WIDE_TILES, _TALL_TILES)
    bool fp8_matrix = false;  // fp8 pools: both products on the fp8 matrix instruction (HKV_PLAN_FP8_MATRIX)
    hkv_decode_plan_params opt{};  // the planner's settings (0 = the library's choice)
    int32_t *d_pages = nullptr, *d_node_req_idx = nullptr, *d_part_count = nullptr;
    std::vector<int32_t> q_rows;  // row of q / out / lse of every row of the plan (empty: row r is row r)
    int32_t *d_q_rows = nullptr;
    bool profiling = false, profiled_run = false;
    hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};  // begin/end of the node kernel, begin/end of the merge
    // several query tokens per request: n_req above counts query rows (requests x tokens_per_req)
    int32_t tokens_per_req = 1;
    // one allocation (d_row_mask), null when tokens_per_req == 1
    unsigned long long *d_row_mask = nullptr;
    int32_t *d_row_leaf = nullptr, *d_row_limit = nullptr;
    // fp32 pools: no work items; every query row walks its own block table (one allocation: d_bt)
    std::vector<int32_t> row_len;
    int32_t max_pages = 0;
    int32_t *d_bt = nullptr, *d_rows_req = nullptr, *d_rows_len = nullptr;
    int32_t row_parts = 1;  // shares that a row's keys are cut into where the caller's workspace has room for their results
    // growing plans (hkv_decode_plan_create_growing): every request's leaf has block slots in node_pages
    // for reserve_tokens more tokens; grow_items holds, per request, the num_kv_heads items of the leaf's
    // last chunk.  Items and block list are re-sent after every append through a ring of pinned buffers.
    int32_t reserve_tokens = 0, appended = 0;
    std::vector<int32_t> grow_items;
    static constexpr int kGrowSlots = 4;
    char *h_grow = nullptr;  // pinned, kGrowSlots x grow_bytes
    char *d_grow = nullptr;  // the same memory as the device addresses it
    int32_t *d_grow_items = nullptr;  // device copy of grow_items (up to 256 requests: updates by a small kernel)
    size_t grow_bytes = 0;   // items + block list as laid out on the device, a multiple of 16
    hipEvent_t grow_free[kGrowSlots] = {};
    bool grow_in_flight[kGrowSlots] = {};
    int grow_next = 0;
};

struct hkv_prefill_plan {
    hkv_pool *pool = nullptr;
    int32_t n_req = 0, num_q_heads = 0, total_q = 0;
    int32_t key_max_pages = 0;   // row length of the caller's block table (pages)
    int32_t max_pages = 0;       // row length of the device table (16-token blocks)
    std::vector<int32_t> cu_q, block_table, kv_len;   // key of the one-shot cache
    std::vector<PrefillTile> tiles;
    std::vector<PrefillTile> pieces;  // small batches: the tiles in pieces of fewer rows, a workgroup each (empty: the tiles)
    void *dev = nullptr;
    PrefillTile *d_tiles = nullptr;
    int32_t *d_block_table = nullptr;
    int32_t *d_rows_req = nullptr, *d_rows_len = nullptr;  // fp32 pools: per new token (one allocation: d_rows_req)
    // fp8 pools: the pages the batch reads are first dequantised into a bf16 scratch pool in the caller's
    // workspace (page i of the scratch = src_pages[i]); the device block table then holds scratch indices.
    std::vector<int32_t> src_pages;
    int32_t *d_src_pages = nullptr;
    unsigned int *d_fallback = nullptr;  // tiles that repeated with a running maximum, over all runs of the plan
    // tiles split along their keys (empty: a workgroup per tile); the partials go to the caller's workspace
    std::vector<PrefillSegment> segments;
    std::vector<int32_t> seg_begin, seg_tile;  // first segment of every worker; the tile a segment was cut from
    std::vector<PrefillSplitTile> split;
    int32_t n_parts = 0;
    PrefillSegment *d_segments = nullptr;
    int32_t *d_seg_begin = nullptr;
    PrefillSplitTile *d_split = nullptr;
};

struct hkv_pool {
    hkv_pool_desc d{};
    // A page of page_size = 16 * S tokens is S consecutive 16-token blocks of the buffers: block
    // page * S + j holds tokens 16 j .. 16 j + 15 of the page.  Everything behind the entry points
    // (work lists, kernels) deals in 16-token blocks; page ids are translated where they come in.
    int32_t blocks_per_page = 1;
    std::vector<int32_t> refcnt;
    std::deque<int32_t> free_list;
    // Staging of page ids for kv_pool_write: a ring of slots (pinned host + device, one allocation
    // each), so that back-to-back writes on a stream do not wait for one another; a slot is reused
    // only after the event recorded behind its last write has completed.
    static constexpr int kMaxWritePages = 65536;
    static constexpr int kWriteSlots = 8;
    int32_t *h_ids = nullptr;  // pinned host, kWriteSlots x kMaxWritePages
    int32_t *hd_ids = nullptr; // the same memory as the device addresses it (source of the copy kernel)
    int32_t *d_ids = nullptr;  // device, same shape
    hipEvent_t slot_free[kWriteSlots] = {};
    bool slot_in_flight[kWriteSlots] = {};
    int next_slot = 0;
    hkv_decode_plan *cached_decode = nullptr;
    hkv_prefill_plan *cached_prefill = nullptr;
};

// ---------------------------------------------------------------------------------------------
extern "C" const char *hkv_last_error(void) { return g_err.c_str(); }

// ---------------------------------------------------------------------------------------------
// pool
extern "C" int kv_pool_create(const hkv_pool_desc *desc, hkv_pool **out) {
    if (!desc || !out) return fail(HKV_EINVAL, "kv_pool_create: null argument");
    *out = nullptr;
    if ((desc->page_size != 16 && desc->page_size != 32 && desc->page_size != 64 && desc->page_size != 128) ||
        desc->head_dim != HKV_HEAD_DIM)
        return fail(HKV_ESHAPE, "kv_pool_create: page_size must be 16, 32, 64 or 128 and head_dim 128 (got %d, %d)",
                    desc->page_size, desc->head_dim);
    if ((int64_t)desc->num_pages * (desc->page_size / HKV_PAGE_SIZE) > INT32_MAX)
        return fail(HKV_EINVAL, "kv_pool_create: too many 16-token blocks");
    if (desc->dtype != HKV_BF16 && desc->dtype != HKV_FP8_E4M3 && desc->dtype != HKV_FP32)
        return fail(HKV_ESHAPE, "kv_pool_create: pool dtype %d (bf16, fp8 e4m3 or fp32)", desc->dtype);
    if (desc->num_pages <= 0 || desc->num_kv_heads <= 0)
        return fail(HKV_EINVAL, "kv_pool_create: num_pages and num_kv_heads must be positive");
    if (!desc->k_pages || !desc->v_pages) return fail(HKV_EINVAL, "kv_pool_create: null page buffer");
    if (desc->dtype == HKV_FP8_E4M3 && (!desc->k_scale || !desc->v_scale))
        return fail(HKV_ESHAPE, "kv_pool_create: fp8 pools need k_scale and v_scale");
    if ((reinterpret_cast<uintptr_t>(desc->k_pages) | reinterpret_cast<uintptr_t>(desc->v_pages)) & 15)
        return fail(HKV_EINVAL, "kv_pool_create: page buffers must be 16-byte aligned");
    hkv_pool *p = new (std::nothrow) hkv_pool;
    if (!p) return fail(HKV_ENOMEM, "kv_pool_create: out of host memory");
    p->d = *desc;
    p->d.free_order = nullptr;
    p->blocks_per_page = desc->page_size / HKV_PAGE_SIZE;
    p->refcnt.assign(desc->num_pages, 0);
    if (desc->free_order) {
        std::vector<char> seen(desc->num_pages, 0);
        for (int i = 0; i < desc->num_pages; ++i) {
            int32_t id = desc->free_order[i];
            if (id < 0 || id >= desc->num_pages || seen[id]) {
                delete p;
                return fail(HKV_EINVAL, "kv_pool_create: free_order is not a permutation (entry %d = %d)", i, id);
            }
            seen[id] = 1;
            p->free_list.push_back(id);
        }
    } else {
        for (int i = 0; i < desc->num_pages; ++i) p->free_list.push_back(i);
    }
    *out = p;
    return HKV_OK;
}

extern "C" int kv_pool_destroy(hkv_pool *pool) {
    if (!pool) return HKV_OK;
    if (pool->cached_decode) hkv_decode_plan_destroy(pool->cached_decode);
    if (pool->cached_prefill) hkv_prefill_plan_destroy(pool->cached_prefill);
    for (hipEvent_t e : pool->slot_free)
        if (e) {
            (void)hipEventSynchronize(e);
            (void)hipEventDestroy(e);
        }
    if (pool->d_ids) (void)hipFree(pool->d_ids);
    if (pool->h_ids) (void)hipHostFree(pool->h_ids);
    delete pool;
    return HKV_OK;
}

extern "C" int kv_pool_alloc(hkv_pool *pool, int32_t n, int32_t *ids_out) {
    if (!pool || n < 0 || (n > 0 && !ids_out)) return fail(HKV_EINVAL, "kv_pool_alloc: bad argument");
    if ((size_t)n > pool->free_list.size())
        return fail(HKV_ENOMEM, "kv_pool_alloc: %d pages requested, %zu free", n, pool->free_list.size());
    for (int i = 0; i < n; ++i) {
        int32_t id = pool->free_list.front();
        pool->free_list.pop_front();
        pool->refcnt[id] = 1;
        ids_out[i] = id;
    }
    return HKV_OK;
}

static int check_held(const hkv_pool *pool, int32_t n, const int32_t *ids, const char *who) {
    if (!pool || n < 0 || (n > 0 && !ids)) return fail(HKV_EINVAL, "%s: bad argument", who);
    for (int i = 0; i < n; ++i) {
        if (ids[i] < 0 || ids[i] >= pool->d.num_pages)
            return fail(HKV_ERANGE, "%s: page id %d (entry %d) outside pool of %d pages", who, ids[i], i,
                        pool->d.num_pages);
    }
    // a page listed k times needs at least k references for a release; at least 1 for a retain
    return HKV_OK;
}

extern "C" int kv_pool_retain(hkv_pool *pool, int32_t n, const int32_t *ids) {
    if (int rc = check_held(pool, n, ids, "kv_pool_retain")) return rc;
    for (int i = 0; i < n; ++i)
        if (pool->refcnt[ids[i]] <= 0) return fail(HKV_EINVAL, "kv_pool_retain: page %d is not allocated", ids[i]);
    for (int i = 0; i < n; ++i) ++pool->refcnt[ids[i]];
    return HKV_OK;
}

extern "C" int kv_pool_release(hkv_pool *pool, int32_t n, const int32_t *ids) {
    if (int rc = check_held(pool, n, ids, "kv_pool_release")) return rc;
    std::vector<int32_t> sorted(ids, ids + n);  // a page may occur several times: count per page
    std::sort(sorted.begin(), sorted.end());
    for (int i = 0, run = 0; i < n; ++i) {
        run = (i > 0 && sorted[i] == sorted[i - 1]) ? run + 1 : 1;
        if (run > pool->refcnt[sorted[i]])
            return fail(HKV_EINVAL, "kv_pool_release: page %d released more often than it is held", sorted[i]);
    }
    for (int i = 0; i < n; ++i)
        if (--pool->refcnt[ids[i]] == 0) pool->free_list.push_back(ids[i]);
    return HKV_OK;
}

extern "C" int32_t kv_pool_num_free(const hkv_pool *pool) {
    if (!pool) return fail(HKV_EINVAL, "kv_pool_num_free: null pool");
    return (int32_t)pool->free_list.size();
}

extern "C" int32_t kv_pool_page_size(const hkv_pool *pool) {
    if (!pool) return fail(HKV_EINVAL, "kv_pool_page_size: null pool");
    return pool->d.page_size;
}

extern "C" int32_t kv_pool_refcount(const hkv_pool *pool, int32_t page_id) {
    if (!pool) return fail(HKV_EINVAL, "kv_pool_refcount: null pool");
    if (page_id < 0 || page_id >= pool->d.num_pages) return fail(HKV_ERANGE, "kv_pool_refcount: page id %d", page_id);
    return pool->refcnt[page_id];
}

static PoolView view_of(const hkv_pool *p) {
    return PoolView{p->d.k_pages, p->d.v_pages, p->d.k_scale, p->d.v_scale, p->d.num_kv_heads, p->d.dtype};
}

extern "C" int kv_pool_copy_on_write(hkv_pool *pool, int32_t n, int32_t *ids, void *stream) {
    if (int rc = check_held(pool, n, ids, "kv_pool_copy_on_write")) return rc;
    std::vector<int32_t> sorted(ids, ids + n);
    std::sort(sorted.begin(), sorted.end());
    size_t shared = 0;
    for (int i = 0; i < n; ++i) {
        if (i > 0 && sorted[i] == sorted[i - 1])
            return fail(HKV_EINVAL, "kv_pool_copy_on_write: page %d listed twice", sorted[i]);
        if (pool->refcnt[sorted[i]] <= 0)
            return fail(HKV_EINVAL, "kv_pool_copy_on_write: page %d is not allocated", sorted[i]);
        shared += pool->refcnt[sorted[i]] > 1;
    }
    if (shared > pool->free_list.size())
        return fail(HKV_ENOMEM, "kv_pool_copy_on_write: %zu private copies needed, %zu pages free", shared,
                    pool->free_list.size());
    PoolCopyLaunch a{};
    a.pool = view_of(pool);
    a.blocks_per_page = pool->blocks_per_page;
    for (int i = 0; i < n; ++i) {
        const int32_t old = ids[i];
        if (pool->refcnt[old] == 1) continue;  // sole holder: it may write in place
        const int32_t fresh = pool->free_list.front();
        pool->free_list.pop_front();
        pool->refcnt[fresh] = 1;
        --pool->refcnt[old];
        ids[i] = fresh;
        a.src[a.n] = old;
        a.dst[a.n] = fresh;
        if (++a.n == kMaxCopyPairs) {
            HKV_HIP(launch_pool_copy(a, static_cast<hipStream_t>(stream)));
            a.n = 0;
        }
    }
    HKV_HIP(launch_pool_copy(a, static_cast<hipStream_t>(stream)));
    return HKV_OK;
}

static int ensure_write_staging(hkv_pool *pool) {
    if (pool->h_ids) return HKV_OK;
    const size_t bytes = sizeof(int32_t) * hkv_pool::kMaxWritePages * hkv_pool::kWriteSlots;
    HKV_HIP(hipHostMalloc((void **)&pool->h_ids, bytes, hipHostMallocDefault));
    HKV_HIP(hipHostGetDevicePointer((void **)&pool->hd_ids, pool->h_ids, 0));
    HKV_HIP(hipMalloc((void **)&pool->d_ids, bytes));
    for (hipEvent_t &e : pool->slot_free) HKV_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    return HKV_OK;
}

extern "C" int kv_pool_write(hkv_pool *pool, const int32_t *page_ids, int32_t first_slot, int32_t n_tokens,
                             const void *k_src, const void *v_src, void *stream) {
    if (!pool) return fail(HKV_EINVAL, "kv_pool_write: null pool");
    const int P = pool->d.page_size, S = pool->blocks_per_page;
    if (n_tokens < 0 || first_slot < 0 || first_slot >= P)
        return fail(HKV_EINVAL, "kv_pool_write: n_tokens %d, first_slot %d", n_tokens, first_slot);
    if (n_tokens == 0) return HKV_OK;
    if (!page_ids || !k_src || !v_src) return fail(HKV_EINVAL, "kv_pool_write: null argument");
    if ((reinterpret_cast<uintptr_t>(k_src) | reinterpret_cast<uintptr_t>(v_src)) & 15)
        return fail(HKV_EINVAL, "kv_pool_write: k_src and v_src must be 16-byte aligned");
    // 16-token blocks touched: b0 .. b1 of the listed pages' concatenated blocks
    const int64_t b0 = first_slot / HKV_PAGE_SIZE, b1 = ((int64_t)first_slot + n_tokens - 1) / HKV_PAGE_SIZE;
    const int64_t n_pg = b1 - b0 + 1;
    if (n_pg > hkv_pool::kMaxWritePages)
        return fail(HKV_EINVAL, "kv_pool_write: %lld pages in one call (limit %d)", (long long)n_pg,
                    hkv_pool::kMaxWritePages);
    for (int64_t i = 0; i <= b1 / S; ++i)
        if (page_ids[i] < 0 || page_ids[i] >= pool->d.num_pages)
            return fail(HKV_ERANGE, "kv_pool_write: page id %d (entry %lld) outside pool of %d pages", page_ids[i],
                        (long long)i, pool->d.num_pages);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (n_pg <= kMaxInlineWrite && pool->d.dtype != HKV_FP32) {  // the ids travel in the kernel arguments: one launch, no staging
        int32_t ids[kMaxInlineWrite];
        for (int64_t b = b0; b <= b1; ++b) ids[b - b0] = page_ids[b / S] * S + (int32_t)(b % S);
        const PoolWriteLaunch a{pool->d.k_pages, pool->d.v_pages, pool->d.k_scale, pool->d.v_scale, pool->d.num_kv_heads, pool->d.dtype,
                                nullptr, (int32_t)n_pg, first_slot % HKV_PAGE_SIZE, n_tokens, k_src, v_src, nullptr, ids};
        HKV_HIP(launch_pool_write(a, s));
        return HKV_OK;
    }
    if (int rc = ensure_write_staging(pool)) return rc;
    const int slot = pool->next_slot;
    pool->next_slot = (slot + 1) % hkv_pool::kWriteSlots;
    if (pool->slot_in_flight[slot]) HKV_HIP(hipEventSynchronize(pool->slot_free[slot]));  // its last write is done
    int32_t *h = pool->h_ids + (size_t)slot * hkv_pool::kMaxWritePages;
    int32_t *d = pool->d_ids + (size_t)slot * hkv_pool::kMaxWritePages;
    for (int64_t b = b0; b <= b1; ++b) h[b - b0] = page_ids[b / S] * S + (int32_t)(b % S);
    // a copy kernel on the stream reads the pinned slot (a DMA copy between kernels of one stream costs more)
    HKV_HIP(launch_upload(pool->hd_ids + (size_t)slot * hkv_pool::kMaxWritePages, d, align_up(sizeof(int32_t) * (size_t)n_pg, 16), s));
    PoolWriteLaunch a{pool->d.k_pages, pool->d.v_pages, pool->d.k_scale, pool->d.v_scale, pool->d.num_kv_heads,
                      pool->d.dtype, d, (int32_t)n_pg, first_slot % HKV_PAGE_SIZE, n_tokens, k_src, v_src, nullptr, nullptr};
    if (pool->d.dtype == HKV_FP32)
        HKV_HIP(launch_pool_write_fp32(a, s));
    else
        HKV_HIP(launch_pool_write(a, s));
    HKV_HIP(hipEventRecord(pool->slot_free[slot], s));
    pool->slot_in_flight[slot] = true;
    return HKV_OK;
}

extern "C" int kv_pool_append(hkv_pool *pool, const int32_t *page_ids, const int32_t *slots, int32_t n,
                              const void *k_src, const void *v_src, void *stream) {
    if (!pool) return fail(HKV_EINVAL, "kv_pool_append: null pool");
    if (n < 0) return fail(HKV_EINVAL, "kv_pool_append: n %d", n);
    if (n == 0) return HKV_OK;
    if (!page_ids || !slots || !k_src || !v_src) return fail(HKV_EINVAL, "kv_pool_append: null argument");
    if (pool->d.dtype == HKV_FP32) return fail(HKV_ESHAPE, "kv_pool_append: bf16 and fp8 pools only");
    if ((reinterpret_cast<uintptr_t>(k_src) | reinterpret_cast<uintptr_t>(v_src)) & 15)
        return fail(HKV_EINVAL, "kv_pool_append: k_src and v_src must be 16-byte aligned");
    if (n > hkv_pool::kMaxWritePages / 2) return fail(HKV_EINVAL, "kv_pool_append: %d tokens in one call (limit %d)", n, hkv_pool::kMaxWritePages / 2);
    const int P = pool->d.page_size, S = pool->blocks_per_page;
    for (int i = 0; i < n; ++i) {
        if (page_ids[i] < 0 || page_ids[i] >= pool->d.num_pages)
            return fail(HKV_ERANGE, "kv_pool_append: page id %d (entry %d) outside pool of %d pages", page_ids[i], i, pool->d.num_pages);
        if (slots[i] < 0 || slots[i] >= P) return fail(HKV_EINVAL, "kv_pool_append: slot %d (entry %d)", slots[i], i);
        if (pool->refcnt[page_ids[i]] > 1)
            return fail(HKV_EINVAL, "kv_pool_append: page %d (entry %d) has %d owners: kv_pool_copy_on_write first", page_ids[i], i,
                        pool->refcnt[page_ids[i]]);
    }
    if (n > 1) {  // two tokens of one call in one block would race on the block's scale and on its re-encoding
        std::vector<int32_t> blocks(n);
        for (int i = 0; i < n; ++i) blocks[i] = page_ids[i] * S + slots[i] / HKV_PAGE_SIZE;
        std::sort(blocks.begin(), blocks.end());
        auto dup = std::adjacent_find(blocks.begin(), blocks.end());
        if (dup != blocks.end())
            return fail(HKV_EINVAL, "kv_pool_append: two tokens go to block %d of page %d", *dup % S, *dup / S);
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (n <= kMaxInlineAppend) {  // the usual decode batch: everything travels in the kernel arguments
        PoolAppendInline a{};
        a.base = PoolWriteLaunch{pool->d.k_pages, pool->d.v_pages, pool->d.k_scale, pool->d.v_scale, pool->d.num_kv_heads,
                                 pool->d.dtype, nullptr, n, 0, n, k_src, v_src, nullptr, nullptr};
        for (int i = 0; i < n; ++i) {
            a.block[i] = page_ids[i] * S + slots[i] / HKV_PAGE_SIZE;
            a.slot[i] = (uint8_t)(slots[i] % HKV_PAGE_SIZE);
        }
        HKV_HIP(launch_pool_append_inline(a, s));
        return HKV_OK;
    }
    if (int rc = ensure_write_staging(pool)) return rc;
    const int slot = pool->next_slot;
    pool->next_slot = (slot + 1) % hkv_pool::kWriteSlots;
    if (pool->slot_in_flight[slot]) HKV_HIP(hipEventSynchronize(pool->slot_free[slot]));
    int32_t *h = pool->h_ids + (size_t)slot * hkv_pool::kMaxWritePages;
    int32_t *d = pool->d_ids + (size_t)slot * hkv_pool::kMaxWritePages;
    for (int i = 0; i < n; ++i) {  // block ids, then the slots inside them
        h[i] = page_ids[i] * S + slots[i] / HKV_PAGE_SIZE;
        h[n + i] = slots[i] % HKV_PAGE_SIZE;
    }
    HKV_HIP(launch_upload(pool->hd_ids + (size_t)slot * hkv_pool::kMaxWritePages, d, align_up(sizeof(int32_t) * 2 * (size_t)n, 16), s));
    PoolWriteLaunch a{pool->d.k_pages, pool->d.v_pages, pool->d.k_scale, pool->d.v_scale, pool->d.num_kv_heads,
                      pool->d.dtype, d, n, 0, n, k_src, v_src, d + n, nullptr};
    HKV_HIP(launch_pool_write(a, s));
    HKV_HIP(hipEventRecord(pool->slot_free[slot], s));
    pool->slot_in_flight[slot] = true;
    return HKV_OK;
}

// ---------------------------------------------------------------------------------------------
// forest
// whole_page_parents: a node with children must hold a multiple of 16 tokens (what a flat block table
// needs: positions along a path then map to pages without gaps); false for callers that walk the forest
// node by node.
static int validate_forest(const hkv_node *nodes, int32_t n_nodes, const int32_t *node_pages, int32_t n_node_pages,
                           const char *who, bool whole_page_parents = true, int page_size = HKV_PAGE_SIZE) {
    if (n_nodes < 0 || n_node_pages < 0 || (n_nodes > 0 && !nodes) || (n_node_pages > 0 && !node_pages))
        return fail(HKV_EINVAL, "%s: bad forest arguments", who);
    std::vector<char> has_child(n_nodes, 0);
    for (int v = 0; v < n_nodes; ++v) {
        const hkv_node &nd = nodes[v];
        if (nd.parent < -1 || nd.parent >= v)
            return fail(HKV_ETREE, "%s: node %d has parent %d (parents must come first)", who, v, nd.parent);
        if (nd.n_tokens < 0 || nd.n_pages != (nd.n_tokens + page_size - 1) / page_size)
            return fail(HKV_ETREE, "%s: node %d has %d tokens but %d pages", who, v, nd.n_tokens, nd.n_pages);
        if (nd.page_begin < 0 || (int64_t)nd.page_begin + nd.n_pages > n_node_pages)
            return fail(HKV_ERANGE, "%s: node %d pages [%d, %d) outside node_pages of %d", who, v, nd.page_begin,
                        nd.page_begin + nd.n_pages, n_node_pages);
        if (nd.parent >= 0) has_child[nd.parent] = 1;
    }
    if (whole_page_parents)
        for (int v = 0; v < n_nodes; ++v)
            if (has_child[v] && nodes[v].n_tokens % page_size)
                return fail(HKV_ETREE, "%s: node %d has children but %d tokens (not a multiple of %d)", who, v,
                            nodes[v].n_tokens, page_size);
    return HKV_OK;
}

static int build_node_req_csr(const hkv_node *nodes, int32_t n_nodes, const int32_t *req_leaf, int32_t n_req,
                              std::vector<int32_t> &indptr, std::vector<int32_t> &idx, const char *who) {
    if (n_req < 0 || (n_req > 0 && !req_leaf)) return fail(HKV_EINVAL, "%s: bad request list", who);
    indptr.assign((size_t)n_nodes + 1, 0);
    for (int r = 0; r < n_req; ++r) {
        if (req_leaf[r] < 0 || req_leaf[r] >= n_nodes)
            return fail(HKV_ERANGE, "%s: request %d ends at node %d of %d", who, r, req_leaf[r], n_nodes);
        for (int v = req_leaf[r]; v >= 0; v = nodes[v].parent) ++indptr[v + 1];
    }
    for (int v = 0; v < n_nodes; ++v) indptr[v + 1] += indptr[v];
    idx.assign((size_t)indptr[n_nodes], 0);
    std::vector<int32_t> fill(indptr.begin(), indptr.end() - 1);
    for (int r = 0; r < n_req; ++r)  // ascending r keeps every node's list sorted
        for (int v = req_leaf[r]; v >= 0; v = nodes[v].parent) idx[fill[v]++] = r;
    return HKV_OK;
}

extern "C" int prefix_tree_flatten(const hkv_node *nodes, int32_t n_nodes, const int32_t *node_pages,
                                   int32_t n_node_pages, const int32_t *req_leaf, int32_t n_req, int32_t max_pages,
                                   int32_t *block_table, int32_t *kv_len, int32_t *node_req_indptr,
                                   int32_t *node_req_idx, int32_t *node_tok_start) {
    return prefix_tree_flatten_paged(nodes, n_nodes, node_pages, n_node_pages, req_leaf, n_req, HKV_PAGE_SIZE, max_pages,
                                     block_table, kv_len, node_req_indptr, node_req_idx, node_tok_start);
}

extern "C" int prefix_tree_flatten_paged(const hkv_node *nodes, int32_t n_nodes, const int32_t *node_pages,
                                         int32_t n_node_pages, const int32_t *req_leaf, int32_t n_req,
                                         int32_t page_size, int32_t max_pages, int32_t *block_table, int32_t *kv_len,
                                         int32_t *node_req_indptr, int32_t *node_req_idx, int32_t *node_tok_start) {
    if (max_pages < 0) return fail(HKV_EINVAL, "prefix_tree_flatten: max_pages %d", max_pages);
    if (page_size != 16 && page_size != 32 && page_size != 64 && page_size != 128)
        return fail(HKV_ESHAPE, "prefix_tree_flatten: page_size %d (16, 32, 64 or 128)", page_size);
    if (int rc = validate_forest(nodes, n_nodes, node_pages, n_node_pages, "prefix_tree_flatten", true, page_size)) return rc;
    std::vector<int32_t> indptr, idx;
    if (int rc = build_node_req_csr(nodes, n_nodes, req_leaf, n_req, indptr, idx, "prefix_tree_flatten")) return rc;
    std::vector<int32_t> tok_start(n_nodes, 0), pages_before(n_nodes, 0);
    for (int v = 0; v < n_nodes; ++v) {
        int par = nodes[v].parent;
        if (par >= 0) {
            tok_start[v] = tok_start[par] + nodes[par].n_tokens;
            pages_before[v] = pages_before[par] + nodes[par].n_pages;
        }
    }
    for (int r = 0; r < n_req; ++r) {
        int leaf = req_leaf[r];
        int total_pages = pages_before[leaf] + nodes[leaf].n_pages;
        if (total_pages > max_pages)
            return fail(HKV_ENOMEM, "prefix_tree_flatten: request %d needs %d pages, max_pages is %d", r, total_pages,
                        max_pages);
    }
    for (int r = 0; r < n_req; ++r) {
        int leaf = req_leaf[r];
        if (kv_len) kv_len[r] = tok_start[leaf] + nodes[leaf].n_tokens;
        if (!block_table) continue;
        int32_t *row = block_table + (size_t)r * max_pages;
        int total_pages = pages_before[leaf] + nodes[leaf].n_pages;
        for (int i = total_pages; i < max_pages; ++i) row[i] = -1;
        for (int v = leaf; v >= 0; v = nodes[v].parent)
            for (int j = 0; j < nodes[v].n_pages; ++j) row[pages_before[v] + j] = node_pages[nodes[v].page_begin + j];
    }
    if (node_req_indptr) memcpy(node_req_indptr, indptr.data(), sizeof(int32_t) * indptr.size());
    if (node_req_idx && !idx.empty()) memcpy(node_req_idx, idx.data(), sizeof(int32_t) * idx.size());
    if (node_tok_start && n_nodes) memcpy(node_tok_start, tok_start.data(), sizeof(int32_t) * n_nodes);
    return HKV_OK;
}

extern "C" int prefix_tree_prefill_usage(const hkv_node *nodes, int32_t n_nodes, const int32_t *calls,
                                         int32_t n_calls, int64_t *u_p) {
    if (n_nodes < 0 || n_calls < 0 || (n_nodes > 0 && !nodes) || (n_calls > 0 && (!calls || !u_p)))
        return fail(HKV_EINVAL, "prefix_tree_prefill_usage: bad argument");
    for (int v = 0; v < n_nodes; ++v)
        if (nodes[v].parent < -1 || nodes[v].parent >= v || nodes[v].n_tokens < 0)
            return fail(HKV_ETREE, "prefix_tree_prefill_usage: node %d malformed", v);
    // depth and token count from the root let two leaves meet at their lowest common ancestor
    std::vector<int32_t> depth(n_nodes, 0);
    std::vector<int64_t> tok_end(n_nodes, 0);
    for (int v = 0; v < n_nodes; ++v) {
        int par = nodes[v].parent;
        depth[v] = par < 0 ? 0 : depth[par] + 1;
        tok_end[v] = (par < 0 ? 0 : tok_end[par]) + nodes[v].n_tokens;
    }
    for (int j = 0; j < n_calls; ++j) {
        if (calls[j] < 0 || calls[j] >= n_nodes)
            return fail(HKV_ERANGE, "prefix_tree_prefill_usage: call %d names node %d of %d", j, calls[j], n_nodes);
        int64_t shared = 0;
        if (j > 0) {
            int a = calls[j - 1], b = calls[j];
            while (a >= 0 && b >= 0 && a != b) {
                if (depth[a] >= depth[b]) a = nodes[a].parent; else b = nodes[b].parent;
            }
            if (a >= 0 && a == b) shared = tok_end[a];
        }
        u_p[j] = tok_end[calls[j]] - shared;
    }
    return HKV_OK;
}

// ---------------------------------------------------------------------------------------------
// lse_merge
extern "C" int lse_merge(const float *o_parts, const float *lse_parts, const int32_t *row_indptr,
                         const int32_t *part_idx, int32_t n_rows, void *out, int32_t out_dtype, float *lse_out,
                         void *stream) {
    if (n_rows < 0) return fail(HKV_EINVAL, "lse_merge: n_rows %d", n_rows);
    if (out_dtype != HKV_BF16 && out_dtype != HKV_FP32) return fail(HKV_ESHAPE, "lse_merge: out_dtype %d", out_dtype);
    if (n_rows == 0) return HKV_OK;
    if (!o_parts || !lse_parts || !row_indptr || !part_idx || !out) return fail(HKV_EINVAL, "lse_merge: null argument");
    if ((reinterpret_cast<uintptr_t>(o_parts) & 7) || (reinterpret_cast<uintptr_t>(out) & 7))
        return fail(HKV_EINVAL, "lse_merge: o_parts and out must be 8-byte aligned");
    HKV_HIP(launch_lse_merge(o_parts, lse_parts, row_indptr, part_idx, n_rows, out, out_dtype, lse_out,
                             static_cast<hipStream_t>(stream)));
    return HKV_OK;
}

extern "C" int lse_merge_dense(const float *o_parts, const float *lse_parts, const int32_t *part_count,
                               int32_t rows_per_count, int32_t max_parts, int32_t n_rows, void *out, int32_t out_dtype,
                               float *lse_out, void *stream) {
    if (n_rows < 0 || rows_per_count <= 0 || max_parts <= 0)
        return fail(HKV_EINVAL, "lse_merge_dense: n_rows %d, rows_per_count %d, max_parts %d", n_rows, rows_per_count,
                    max_parts);
    if (out_dtype != HKV_BF16 && out_dtype != HKV_FP32) return fail(HKV_ESHAPE, "lse_merge_dense: out_dtype %d", out_dtype);
    if (n_rows == 0) return HKV_OK;
    if (!o_parts || !lse_parts || !part_count || !out) return fail(HKV_EINVAL, "lse_merge_dense: null argument");
    if ((reinterpret_cast<uintptr_t>(o_parts) | reinterpret_cast<uintptr_t>(out)) & 15)
        return fail(HKV_EINVAL, "lse_merge_dense: o_parts and out must be 16-byte aligned");
    HKV_HIP(launch_lse_merge_dense(o_parts, lse_parts, part_count, rows_per_count, max_parts, n_rows, out, out_dtype,
                                   lse_out, static_cast<hipStream_t>(stream)));
    return HKV_OK;
}

// Room for so many partials: o as fp16, lse, and the factor each one is to be multiplied by.
static size_t partials_bytes(int64_t n) {
    return align_up((size_t)n * HKV_HEAD_DIM * sizeof(uint16_t), 256) + 2 * align_up((size_t)n * sizeof(float), 256);
}

// ---------------------------------------------------------------------------------------------
// decode planning
//
// A node with T tokens that R requests pass through is cut into work items of at most 64 (tall tiles: 128) query
// rows (R_item * G) and a token chunk each.  Every item yields one partial result per row, so the
// chunk length trades parallelism (more items) against partial-result traffic (516 B per row and
// item, written once and read once).
//
// Partials are stored densely: the path above a node is common to every request below it, so the
// chunks of a node get the same positions k in the partial lists of all those requests, and row
// (r, h) keeps its partials at (r*Hq + h)*max_parts + k.  The merge then needs no index lists,
// only the number of partials per request.
//
static void plan_items(hkv_decode_plan &pl) {
    const int G = pl.group;
    const int Hkv = pl.pool->d.num_kv_heads;
    const int n_nodes = (int)pl.nodes.size();
    const hkv_decode_plan_params &opt = pl.opt;
    auto or_default = [](int32_t v, int dflt) { return v != 0 ? (int)v : dflt; };
    const ChipShape chip = chip_shape();
    const int max_req_per_item = std::max(1, or_default(opt.max_rows, pl.tile_form == 2 ? 128 : 64) / G);
    // Chunk lengths.  Nodes read by at most 16 rows ("leaf type") stay whole unless the forest has
    // fewer (node, head) units than workgroups fit on the chip at once; then they are cut, but not
    // below 256 tokens.  Nodes shared by more rows get chunks near the typical leaf-type item, so that
    // both kinds finish together; for 32-row tiles that length is where the search below begins.
    // Nodes shared by many rows go to the 256-row tile kernel (not when the caller asked for the fp8 matrix instruction).
    const int tile_min_rows = or_default(opt.tile_min_rows, 128);
    // The second kernel, its stream and the two events pay only when that share of the step is large (measured:
    // c2 and c3, 2 and 9 GFLOP of such work in steps of 30 to 50 us, lose; c5, 137 GFLOP in 0.5 ms, gains 11 %).
    // Plans with several query tokens per request: the tile kernel knows no per-row visibility, but only the requests'
    // last nodes need it; every other node is seen whole by all rows below it.  There the tiles run in front of the other
    // items' kernel on all compute units; without them a root of 64 requests x 21 drafted tokens x 4 heads reads its K/V
    // from L2 84 times, once per 64 rows.  fp8 pools, tokens of the shared node x requests x drafted tokens, work of the
    // tiles, step without -> with them: 1024 x 64 x 21, 23 GFLOP, 86.4 -> 79.5 us; 2048 x 64 x 8, 17 GFLOP, 52.3 -> 58.5 (the
    // second kernel's ramp); 4096 x 64 x 8, 34 GFLOP, 75.2 -> 72.2; 8192 x 32 x 8, 34 GFLOP, 62.4 -> 63.3; 2048 x 64 x 21,
    // 45 GFLOP, 114.7 -> 100.4; 8192 x 64 x 4 x 8 heads, 69 GFLOP, 119 -> 100.6.  Below 30 GFLOP the shapes that lose lose more
    // than the others gain.  Only beside last nodes of more than 16 rows: in one launch with smaller ones (4 tokens x 4
    // heads, 17 GFLOP) it lost too (39.0 -> 46.2 us).
    // bf16 pools only if the caller asks (tile_min_gflop): the tile keeps one reference per row, so that the heaviest
    // probabilities lie anywhere in their binade when they are rounded to bf16, and the error against 64 bits grows from
    // 0.00217 to 0.00231 (64 x 21 over 2048 + 512 tokens, 122 -> 97 us).  With fp8 pools the V scale comes in before that
    // rounding, whatever the reference, and the error is the same (0.00236).
    std::vector<char> row_node(n_nodes, 0);  // nodes whose tokens some rows see in part
    bool wide_row_node = false;
    if (pl.row_visibility)
        for (int r = 0; r < pl.n_req; ++r) {
            const int v = pl.req_leaf[r];
            row_node[v] = 1;
            wide_row_node = wide_row_node || (pl.node_req_indptr[v + 1] - pl.node_req_indptr[v]) * G > 16;
        }
    bool tiles_pay = false;
    {
        double flop = 0;
        for (int v = 0; v < n_nodes; ++v) {
            const int R = pl.node_req_indptr[v + 1] - pl.node_req_indptr[v];
            if (!row_node[v] && R * G >= std::max(tile_min_rows, kMinTileItemRows))
                flop += 4.0 * HKV_HEAD_DIM * pl.nodes[v].n_tokens * (double)R * pl.num_q_heads;
        }
        if (pl.row_visibility)
            tiles_pay = wide_row_node && (opt.tile_min_gflop > 0 ? flop >= 1e9 * opt.tile_min_gflop : pl.pool->d.dtype == HKV_FP8_E4M3 && flop >= 30e9);
        else
            tiles_pay = opt.tile_min_gflop < 0 || flop >= 1e9 * or_default(opt.tile_min_gflop, 40);
    }
    auto tiled = [&](int v) {
        const int R = pl.node_req_indptr[v + 1] - pl.node_req_indptr[v];
        return tiles_pay && !row_node[v] && !pl.fp8_matrix && pl.nodes[v].n_tokens > 0 &&
               R * G >= std::max(tile_min_rows, kMinTileItemRows);
    };
    const bool fp8_pool = pl.pool->d.dtype == HKV_FP8_E4M3;
    // The tile kernel's share of the chip: its persistent workgroups hold one compute unit each for as long as
    // the other kernel streams its bytes, so their number follows from the two amounts of work (matrix
    // arithmetic at about 3.5 TFLOP/s per compute unit against bytes at about 5.5 TB/s for the chip).
    const int req_per_tile = std::max(1, 256 / G);
    const bool tiles_first = pl.row_visibility;
    if (tiles_first) pl.concurrent = false;
    pl.tile_items.clear();
    pl.tile_workgroups = 0;
    int tile_chunk = kMaxTileItemTokens;
    double step_seconds = 0;  // what streaming all the bytes of the step takes
    {
        double tile_flop = 0, other_bytes = 0, tile_bytes = 0;
        int64_t tile_units = 0, tile_tokens_max = 0;
        const double bytes_per_token = 2.0 * HKV_HEAD_DIM * (fp8_pool ? 1 : 2);
        for (int v = 0; v < n_nodes; ++v) {
            const int R = pl.node_req_indptr[v + 1] - pl.node_req_indptr[v];
            if (pl.nodes[v].n_tokens == 0 || R == 0) continue;
            if (tiled(v)) {
                tile_flop += 4.0 * HKV_HEAD_DIM * pl.nodes[v].n_tokens * (double)R * pl.num_q_heads;
                tile_units += (int64_t)((R + req_per_tile - 1) / req_per_tile) * Hkv;
                tile_tokens_max = std::max<int64_t>(tile_tokens_max, pl.nodes[v].n_tokens);
                tile_bytes += bytes_per_token * pl.nodes[v].n_tokens * Hkv;
            } else {
                other_bytes += bytes_per_token * pl.nodes[v].n_tokens * Hkv;
            }
        }
        step_seconds = (other_bytes + tile_bytes) / 5.6e12;
        if (tile_units > 0) {
            const int n_cu = chip.n_cu;
            int wgs = n_cu;
            if (other_bytes > 0) {
                const double t_other = other_bytes / 5.5e12;
                wgs = (int)(tile_flop / (3.5e12 * t_other) + 0.999);
                wgs = std::min(n_cu - 64, std::max(8, (wgs + 7) / 8 * 8));  // whole groups of 8: one per XCD
            }
            if (tiles_first) wgs = n_cu;
            wgs = std::min(n_cu, or_default(opt.tile_workgroups, wgs));
            pl.tile_workgroups = wgs;
            // chunks: about one item per workgroup (a workgroup that is done gives its compute unit to the other
            // items, and every chunk costs every row below the node a partial), more where the nodes are few
            int64_t n_chunks = std::max<int64_t>(1, std::min<int64_t>((wgs + tile_units / 2) / tile_units, tile_tokens_max / 256));
            if (tiles_first) {  // rounds of items at 1.45 us per 64 tokens and 4 us each, and what the partials cost
                double best_us = 1e30;
                for (int64_t n = (tile_tokens_max + kMaxTileItemTokens - 1) / kMaxTileItemTokens; n <= 8; ++n) {
                    const int64_t blocks = (tile_tokens_max + 64 * n - 1) / (64 * n);
                    const double us = (double)((tile_units * n + wgs - 1) / wgs) * (4.0 + 1.45 * blocks) + (double)n * pl.n_req * pl.num_q_heads * 264 * 2 / 4e6;
                    if (us < best_us) {
                        best_us = us;
                        n_chunks = n;
                    }
                }
            }
            int64_t ch = ((tile_tokens_max + n_chunks - 1) / n_chunks + 63) / 64 * 64;
            tile_chunk = (int)std::min<int64_t>(kMaxTileItemTokens, std::max<int64_t>(256, ch));
            tile_chunk = std::min(kMaxTileItemTokens, or_default(opt.tile_chunk, tile_chunk)) / 16 * 16;
        }
    }
    auto tile_pages = [&](int v) {  // of a chunk of a node that the tile kernel runs: equal chunks of whole blocks
        const int n_chunks = (pl.nodes[v].n_tokens + tile_chunk - 1) / tile_chunk;
        return (pl.nodes[v].n_pages + n_chunks - 1) / n_chunks;
    };
    bool any_shared = false, any_tiled = false;
    int most_req = 0;  // requests below a shared node
    double through = 0, unique = 0, few_tokens = 0;  // K/V tokens: of shared nodes through workgroups / from HBM, of the others
    for (int v = 0; v < n_nodes; ++v) {
        const int R = pl.node_req_indptr[v + 1] - pl.node_req_indptr[v];
        any_tiled = any_tiled || (R > 0 && tiled(v));
        if (pl.nodes[v].n_tokens == 0 || R == 0 || tiled(v)) continue;
        if (R * G > 16) {
            any_shared = true;
            most_req = std::max(most_req, R);
            through += (double)pl.nodes[v].n_tokens * ((R + max_req_per_item - 1) / max_req_per_item);
            unique += pl.nodes[v].n_tokens;
        } else {
            few_tokens += pl.nodes[v].n_tokens;
        }
    }
    const int kNodeGroups = chip.n_cu * (fp8_pool ? 2 : 3);  // workgroups the chip holds at once without shared::body (with it: two per compute unit)
    int64_t leaf_units = 0, leaf_tokens = 0, shared_units = 0;
    for (int v = 0; v < n_nodes; ++v) {
        int R = pl.node_req_indptr[v + 1] - pl.node_req_indptr[v];
        if (pl.nodes[v].n_tokens == 0 || R == 0 || tiled(v)) continue;
        if (R * G > 16) {  // counted at the smallest chunk length used for such nodes
            shared_units += (int64_t)((R + max_req_per_item - 1) / max_req_per_item) * Hkv *
                            ((pl.nodes[v].n_tokens + 511) / 512);
        } else {
            leaf_units += Hkv;
            leaf_tokens += pl.nodes[v].n_tokens;
        }
    }
    int leaf_split = 1;
    if (leaf_units > 0 && leaf_units + shared_units < kNodeGroups / 2)
        leaf_split = (int)((kNodeGroups / 2 + leaf_units - 1) / leaf_units);
    const int mean_leaf = leaf_units ? (int)(leaf_tokens * Hkv / leaf_units) : 512;
    int leaf_chunk = std::max(256, (mean_leaf / leaf_split + 15) / 16 * 16);
    if (leaf_split == 1) leaf_chunk = 1 << 30;  // whole nodes
    int base_chunk = std::min(kMaxSharedItemTokens, std::max(512, std::min(mean_leaf, leaf_chunk) / 16 * 16));
    // The default length; `estimate` below knows when another one is better.  Long shared paths: every chunk costs each row below it one partial (written once, read once) and
    // every item a start-up, while a long item is the last to finish; measured on forests with 2k to 9k
    // shared tokens the best chunk is about a sixth of the path, between 512 and 1024 tokens.  Beyond
    // 16k shared tokens the chunks grow further so that a row collects about 16 partials at most.
    int64_t longest = 0;  // most shared tokens on one path
    {
        std::vector<int64_t> shared_above(n_nodes, 0);
        for (int v = 0; v < n_nodes; ++v) {
            const int R = pl.node_req_indptr[v + 1] - pl.node_req_indptr[v];
            const int64_t up = pl.nodes[v].parent >= 0 ? shared_above[pl.nodes[v].parent] : 0;
            shared_above[v] = up + (R * G > 16 && !tiled(v) ? pl.nodes[v].n_tokens : 0);
            longest = std::max(longest, shared_above[v]);
        }
        int64_t by_path = std::min<int64_t>(1024, (longest / 6 + 128) / 256 * 256);
        if (longest > 16 * by_path) by_path = std::min<int64_t>(kMaxSharedItemTokens, (longest / 16 + 255) / 256 * 256);
        base_chunk = std::max(base_chunk, (int)by_path);
    }
    const int default_chunk = base_chunk;
    leaf_chunk = or_default(opt.leaf_chunk, leaf_chunk) / 16 * 16;
    base_chunk = std::min(kMaxSharedItemTokens, or_default(opt.shared_chunk, base_chunk)) / 16 * 16;
    // Few-row nodes a little longer than what one wavefront takes alone (pack_tokens): run whole, their
    // four wavefronts get only a few steps each and pay a start-up and a combine through LDS for them.
    // When cutting them into pieces of at most pack_tokens makes the forest large enough for the
    // four-items-per-workgroup mode, each wavefront streams a piece of 8 to 12 steps on its own instead
    // (c2: 512-token leaves as 2 x 256, per-node kernel 31.7 -> 30.0 us).  Nodes of 8 / 3 pack_tokens and
    // more keep their four wavefronts: those already get that many steps each.
    const int step_tokens = pl.pool->d.dtype == HKV_FP8_E4M3 ? 64 : 32;
    const int pack_tokens = or_default(opt.pack_tokens, 12 * step_tokens);
    const int pack_mode = or_default(opt.pack, 2);  // 1: never, 2: when the items exceed the resident workgroups, 3: always
    auto cut_for_packing = [&](int n_tokens) { return n_tokens > pack_tokens && 3 * n_tokens < 8 * pack_tokens; };
    // What depends on whether shared nodes run in shared::body (`wide`) or as 16-row tiles.
    struct Layout {
        bool wide;
        int slots;                     // workgroups the chip holds at once
        bool cut_leaves, cut_to_fill;  // few-row nodes cut for packing; only to fill slots
        int shared_chunk, piece_tokens;
        int max_req;                   // requests of an item: up to 64 rows, with tall tiles (tall_body.h) up to 128
    };
    // cut_more: nodes of few rows may be cut only to fill workgroup slots.
    auto lay_out_anew = [&](const bool wide, const bool cut_more) {
        Layout lay{wide, wide ? 2 * chip.n_cu : kNodeGroups, false, false, base_chunk, pack_tokens, max_req_per_item};
        if (leaf_split == 1 && pack_mode != 1 && opt.leaf_chunk == 0) {
            int64_t units = shared_units;
            bool any = false;
            for (int v = 0; v < n_nodes; ++v) {
                const int R = pl.node_req_indptr[v + 1] - pl.node_req_indptr[v];
                const int T = pl.nodes[v].n_tokens;
                if (T == 0 || R == 0 || R * G > 16) continue;
                any |= cut_for_packing(T);
                units += (int64_t)Hkv * (cut_for_packing(T) ? (T + pack_tokens - 1) / pack_tokens : 1);
            }
            const bool beyond_chip = pack_mode == 3 || units > kNodeGroups;
            lay.cut_leaves = any && (beyond_chip || (cut_more && units > lay.slots));
            lay.cut_to_fill = lay.cut_leaves && !beyond_chip;
        }
        // Items of more than 16 rows: how long a chunk?  Such an item costs a start-up, a hand-over between its wavefronts and
        // a partial per row (6 us together) beside 0.8 us per 64 tokens alone and 1.1 to 2.9 us on a full chip (from L2 / from
        // HBM); two run on a compute unit, dispatched in front of the others, which fill what they leave free.  So a chunk
        // that puts a few items into a second round, or leaves the others no room beside the first, costs a whole further
        // item: 4096 tokens x 512 rows + 8 x 1024 x 64 + 128 private leaves, bf16, takes 45 us cut into 768 tokens (512 such
        // items), 34 us at 1024 (320), 39 us at 1376 (256).  From the length above up to the longest there is, the one with
        // the shortest estimated step is taken.
        if (wide && !pl.fp8_matrix && opt.shared_chunk == 0 && opt.leaf_chunk == 0) {
            const bool fp8 = fp8_pool;
            const int64_t slots = lay.slots;
            double other_steps = 0;
            int64_t other_units = 0, rows_below = 0;
            // The searches below look at each length once, however many nodes have it (a walk over all nodes for every candidate
            // made plans of a few hundred nodes take twice as long to create): items a shared node of so many tokens has per
            // chunk, summed; few-row nodes of so many tokens.
            std::vector<std::pair<int32_t, int64_t>> shared_lengths;
            std::vector<int32_t> few_lengths(pack_tokens + 1, 0);
            int64_t few_longer = 0;
            {
                std::vector<int64_t> by_length(kMaxSharedItemTokens + 1, 0);
                for (int v = 0; v < n_nodes; ++v) {
                    const int R = pl.node_req_indptr[v + 1] - pl.node_req_indptr[v], T = pl.nodes[v].n_tokens;
                    if (T == 0 || R == 0 || tiled(v)) continue;
                    if (R * G > 16) {
                        rows_below = std::max<int64_t>(rows_below, (int64_t)R * pl.num_q_heads);
                        const int64_t items = (int64_t)((R + max_req_per_item - 1) / max_req_per_item) * Hkv;
                        if (T <= kMaxSharedItemTokens)
                            by_length[T] += items;
                        else
                            shared_lengths.push_back({T, items});
                    } else {
                        const int pieces = lay.cut_leaves && cut_for_packing(T) ? (T + pack_tokens - 1) / pack_tokens : 1;
                        other_units += (int64_t)pieces * Hkv;
                        other_steps += (double)Hkv * ((T + step_tokens - 1) / step_tokens);
                        if (T <= pack_tokens)
                            ++few_lengths[T];
                        else
                            ++few_longer;
                    }
                }
                for (int T = 1; T <= kMaxSharedItemTokens; ++T)
                    if (by_length[T]) shared_lengths.push_back({T, by_length[T]});
            }
            const double us_alone = 0.8, us_full = std::max(fp8 ? 1.25 : 1.1, (fp8 ? 1.54 : 2.9) * unique / through);  // per 64 tokens
            const bool packs = pack_mode == 3 || (pack_mode == 2 && other_units + shared_units > lay.slots);
            const int64_t other_wgs = packs ? (other_units + 3) / 4 : other_units;
            const double other_us = other_units ? 5.0 + other_steps / other_units / (packs ? 1 : 4) : 1.0;
            int best = lay.shared_chunk;
            double best_us = 1e30;
            int64_t best_n = 0;  // such items at the chunk taken
            for (int ch = lay.shared_chunk; ch <= kMaxSharedItemTokens; ch += 64) {
                int64_t n = 0, longest_blocks = 0;
                for (const auto &[T, items] : shared_lengths) {
                    const int chunks = T <= ch ? 1 : (T + ch - 1) / ch;
                    n += items * chunks;
                    longest_blocks = std::max<int64_t>(longest_blocks, chunks == 1 ? (T + 63) / 64 : (T + 64 * chunks - 1) / (64 * chunks));
                }
                const int64_t full = n / slots, rest = n % slots;
                const double last = rest ? 6.0 + longest_blocks * (us_alone + std::max(0.0, us_full - us_alone) * rest / slots) : 0.0;
                double us = full * (6.0 + longest_blocks * us_full) + last;
                if (other_wgs > 0) {  // in the slots left free, then in all of them
                    const int64_t beside = rest ? (slots - rest) * std::max<int64_t>(1, (int64_t)(last / other_us)) : 0;
                    us = other_wgs <= beside ? std::max(us, other_us) : us + other_us * std::ceil((double)(other_wgs - beside) / slots);
                }
                us += rows_below * 264.0 * 2 / 4e6 * ((longest + ch - 1) / ch);  // the partials, written and read at about 4 TB/s
                if (us < best_us - 1e-9) {
                    best_us = us;
                    best = ch;
                    best_n = n;
                }
            }
            lay.shared_chunk = best;
            // Where both kinds together leave workgroup slots empty, packed nodes that are whole so far are cut until they fill
            // them (a wavefront that streams a node alone is the longest chain of such a launch; below 160 resp. 256 tokens its
            // start-up takes over).  64 requests of 512 private tokens below 4096 shared ones, fp8: 28.9 us whole, 22.8 us as
            // 2 x 256; a few blocks too many and it is 10 % slower.
            if (cut_more && packs && !lay.cut_leaves && best_n + other_wgs < slots)
                for (int piece = std::max(160, 4 * step_tokens); piece < pack_tokens; piece += 16) {
                    int64_t units = 4 * few_longer;
                    for (int T = 1; T <= pack_tokens; ++T)
                        if (few_lengths[T]) units += (int64_t)few_lengths[T] * ((T + piece - 1) / piece);
                    units *= Hkv;
                    if (best_n + (units + 3) / 4 <= slots) {
                        lay.piece_tokens = piece;
                        break;
                    }
                }
        }
        return lay;
    };
    Layout laid_out[2][2];
    bool is_laid_out[2][2] = {};
    auto lay_out = [&](const bool wide, const bool cut_more) {
        if (!is_laid_out[wide][cut_more]) laid_out[wide][cut_more] = lay_out_anew(wide, cut_more);
        is_laid_out[wide][cut_more] = true;
        return laid_out[wide][cut_more];
    };
    struct Cuts {
        int n_chunks, per_chunk;  // blocks of a chunk; the last one may be shorter
    };
    auto cuts_of = [&](const Layout &lay, int T, int R) {  // equal chunks of whole blocks
        int chunk = std::max(16, R * G > 16 ? lay.shared_chunk : leaf_chunk);
        if (R * G <= 16 && ((lay.cut_leaves && cut_for_packing(T)) || (lay.piece_tokens < pack_tokens && T <= pack_tokens)))
            chunk = lay.piece_tokens;  // equal pieces
        const int blocks = (T + HKV_PAGE_SIZE - 1) / HKV_PAGE_SIZE, most = (T + chunk - 1) / chunk, per_chunk = (blocks + most - 1) / most;
        return Cuts{(blocks + per_chunk - 1) / per_chunk, per_chunk};
    };
    // The estimates below look at up to 21 layouts.  Shared nodes of one length below the same number of requests are counted
    // once; `above`: the next shared node on the way up (-1: none).
    struct NodeClass {
        int32_t tokens, n_req, count;
    };
    struct SharedNode {
        int32_t cls, above;
    };
    std::vector<NodeClass> classes;
    std::vector<SharedNode> shared_nodes;
    std::vector<int32_t> shared_at(any_shared ? n_nodes : 0);  // the last shared node down to a node (-1: none)
    if (any_shared) {
        std::vector<std::pair<int64_t, int32_t>> keys;
        for (int v = 0; v < n_nodes; ++v) {
            const int R = pl.node_req_indptr[v + 1] - pl.node_req_indptr[v];
            shared_at[v] = pl.nodes[v].parent >= 0 ? shared_at[pl.nodes[v].parent] : -1;
            if (pl.nodes[v].n_tokens == 0 || R * G <= 16 || tiled(v)) continue;
            keys.push_back({((int64_t)pl.nodes[v].n_tokens << 32) | R, (int32_t)shared_nodes.size()});
            shared_nodes.push_back({0, shared_at[v]});
            shared_at[v] = (int32_t)shared_nodes.size() - 1;
        }
        std::sort(keys.begin(), keys.end());
        for (size_t i = 0; i < keys.size(); ++i) {
            if (i == 0 || keys[i].first != keys[i - 1].first) classes.push_back({(int32_t)(keys[i].first >> 32), (int32_t)(keys[i].first & 0xFFFFFFFF), 0});
            ++classes.back().count;
            shared_nodes[keys[i].second].cls = (int32_t)classes.size() - 1;
        }
    }
    // The other nodes, the same at every chunk length: items of few rows by 32-token steps and by whether one wavefront may
    // take them alone; chunks on the longest path down to the last node without (entry 0) and below each shared one.
    struct FewItems {
        int32_t steps;
        bool packable;
        double n;
    };
    struct Others {
        bool cut_leaves;
        int32_t piece_tokens;
        std::vector<FewItems> few;
        double n_few;
        std::vector<int32_t> chunks;
    };
    std::vector<Others> known;
    auto others_of = [&](const Layout &lay) -> const Others & {
        for (const Others &o : known)
            if (o.cut_leaves == lay.cut_leaves && o.piece_tokens == lay.piece_tokens) return o;
        Others o{lay.cut_leaves, lay.piece_tokens, {}, 0, std::vector<int32_t>(shared_nodes.size() + 1, 0)};
        std::vector<int32_t> chunks_to(n_nodes), count[2];
        for (int v = 0; v < n_nodes; ++v) {
            const int R = pl.node_req_indptr[v + 1] - pl.node_req_indptr[v], T = pl.nodes[v].n_tokens;
            chunks_to[v] = pl.nodes[v].parent >= 0 ? chunks_to[pl.nodes[v].parent] : 0;
            if (T > 0 && R > 0) {
                if (tiled(v)) {
                    chunks_to[v] += (pl.nodes[v].n_pages + tile_pages(v) - 1) / tile_pages(v);
                } else if (R * G <= 16) {
                    const Cuts cut = cuts_of(lay, T, R);
                    const int tokens = std::min(T, cut.per_chunk * HKV_PAGE_SIZE), steps = (tokens + 31) / 32;
                    std::vector<int32_t> &c = count[tokens <= pack_tokens];
                    if ((int)c.size() <= steps) c.resize(steps + 1);
                    c[steps] += cut.n_chunks;
                    chunks_to[v] += cut.n_chunks;
                }
            }
            int32_t &most = o.chunks[any_shared ? shared_at[v] + 1 : 0];
            most = std::max(most, chunks_to[v]);
        }
        for (int packable = 0; packable < 2; ++packable)
            for (size_t steps = 0; steps < count[packable].size(); ++steps)
                if (count[packable][steps]) {
                    o.few.push_back({(int32_t)steps, packable != 0, (double)count[packable][steps] * Hkv});
                    o.n_few += o.few.back().n;
                }
        known.push_back(std::move(o));
        return known.back();
    };
    // A layout's step, us: three times that run beside each other (as a 3-norm), and what the partials cost.  Latency: the
    // workgroups, longest first, on the chip's slots, stretched on a full chip.  Issue, per compute unit: per 64 tokens of an item
    // and active row tile, and per workgroup.  Memory: the nodes' bytes once, and those that items of shared nodes take
    // from L2.  Coefficients: of 27 700 timings (1675 random decode and verification plans, 5 to 250 us, each in both
    // forms and with chunks of 128 to 2048 tokens, three sets of inputs in turn), 7 % rms.
    struct Coefficients {
        double many0, many1, tall;        // a workgroup with an item of a shared node, 64 rows: + per 64 (32-row tiles) or 32 tokens (16-row tiles); less
                                          // by `tall` of that for the share of the rows it does not have
        double few0, few1, pack0, pack1;  // of few rows: + per 128 tokens; a wavefront with one of its own: + per 32
        double full;                      // all that times 1 + full on a full chip
        double block, tile, few_block, wg;
        double mem_shared, mem_few, l2;   // us per MB
        double part, row, base;           // per million partials and rows; launches
    };
    static const Coefficients kBf16Narrow{1.08, 0.616, 0.230, 1.50, 1.25, 0.01, 1.03, 0.162, 0.046, 0.117, 0.477, 0.12, 0.141, 0.164, 0.032, 171, 2.3, 6.7};
    static const Coefficients kBf16Wide{2.53, 0.909, 0.163, 2.37, 1.18, 1.06, 0.92, 0.154, 0.018, 0.166, 0.288, 1.46, 0.134, 0.163, 0.044, 171, 0.6, 6.1};
    static const Coefficients kFp8{1.69, 0.830, 0.155, 2.51, 0.81, 1.39, 0.76, 0.123, 0.047, 0.189, 0.363, 1.49, 0.116, 0.159, 0.070, 175, 1.5, 7.1};
    // Tall tiles (items of up to 128 rows; shorter ones beside them run in shared::body): 8700 timings of 1100 plans of this kind, 5 % rms.
    static const Coefficients kBf16Tall{4.34, 1.01, 0.126, 4.48, 1.47, 3.16, 0.937, 0.103, 0.00341, 0.236, 0.69, 2.69, 0.125, 0.142, 0.0621, 94.1, 0.802, 5.15};
    // Of bf16 plans in the two forms at the length above (1376 plans, 8 % rms), for the choice of the form at that length: closer
    // there than the sets that also know the other lengths (with those 45 of 900 plans lose more than 3 % instead of 28).  They know
    // an item by its length alone.
    static const Coefficients kNarrowThere{0.98, 0.53, 0, 2.48, 0.86, 0.01, 0.31, 0.54, 0.55, 0, 0.68, 1.42, 0.182, 0.141, 0, 84.5, 0, 7.5};
    static const Coefficients kWideThere{1.60, 0.82, 0, 2.48, 0.86, 2.78, 0.24, 0.40, 0.52, 0, 0.36, 2.65, 0.182, 0.154, 0, 84.5, 0, 7.5};
    // Partials per row of a layout (every row has a slot for as many as the longest list holds): chunks on the longest path.
    std::vector<int32_t> class_chunks(classes.size()), shared_chunks_to(shared_nodes.size());
    auto parts_of = [&](const Layout &lay) {
        const Others &others = others_of(lay);
        for (size_t c = 0; c < classes.size(); ++c) class_chunks[c] = cuts_of(lay, classes[c].tokens, classes[c].n_req).n_chunks;
        int32_t parts = std::max(1, others.chunks[0]);
        for (size_t i = 0; i < shared_nodes.size(); ++i) {
            const SharedNode &n = shared_nodes[i];
            shared_chunks_to[i] = (n.above >= 0 ? shared_chunks_to[n.above] : 0) + class_chunks[n.cls];
            parts = std::max(parts, shared_chunks_to[i] + others.chunks[i + 1]);
        }
        return parts;
    };
    auto estimate_by = [&](const Layout &lay, int parts, const Coefficients &k) {
        const double token_mb = 2.0 * HKV_HEAD_DIM * (fp8_pool ? 1 : 2) * 1e-6;  // of one head
        const int tile_rows = lay.wide ? 32 : 16;
        const Others &others = others_of(lay);
        double n_items = others.n_few;
        for (const NodeClass &c : classes)
            n_items += (double)cuts_of(lay, c.tokens, c.n_req).n_chunks * c.count * Hkv * ((c.n_req + lay.max_req - 1) / lay.max_req);
        const bool packs = pack_mode == 3 || (pack_mode == 2 && n_items > lay.slots);
        constexpr int kBins = 512;  // durations in steps of 0.25 us
        double bins[kBins] = {}, n_wgs = 0, work = 0, longest_us = 0, issue = 0, memory = few_tokens * Hkv * token_mb * k.mem_few;
        int top = 0;
        auto add = [&](double wgs, double us) {
            n_wgs += wgs;
            work += wgs * us;
            longest_us = std::max(longest_us, us);
            const int bin = std::min(kBins - 1, (int)(us * 4));
            bins[bin] += wgs;
            top = std::max(top, bin);
        };
        auto add_few = [&](double n, int steps, bool packed) {
            issue += n * ((steps + 1) / 2) * k.few_block;
            packed ? add(0.25 * n, k.pack0 + k.pack1 * steps) : add(n, k.few0 + k.few1 * ((steps + 3) / 4));
        };
        auto add_many = [&](double n, int tokens, int rows) {
            const int blocks = (tokens + 63) / 64, steps = (tokens + 31) / 32;
            issue += n * blocks * (k.block + k.tile * ((rows + tile_rows - 1) / tile_rows));
            memory += n * tokens * token_mb * k.l2;
            add(n, (k.many0 + k.many1 * (lay.wide ? blocks : steps)) * (1.0 + k.tall * (rows / 64.0 - 1.0)));
        };
        for (const FewItems &f : others.few) add_few(f.n, f.steps, packs && f.packable);
        for (const NodeClass &c : classes) {
            const int T = c.tokens, R = c.n_req;
            const Cuts cut = cuts_of(lay, T, R);
            const int tokens = std::min(T, cut.per_chunk * HKV_PAGE_SIZE);
            const double n = (double)c.count * cut.n_chunks * Hkv;
            memory += (double)c.count * T * Hkv * token_mb * k.mem_shared;
            const int groups = (R + lay.max_req - 1) / lay.max_req, rest = R - (groups - 1) * lay.max_req;
            if (k.tile > 0 && !lay.wide && !fp8_pool && groups > 1 && rest * G <= 16) {  // (the remainder beside 16-row tiles, as below)
                add_many(n * (groups - 1), tokens, lay.max_req * G);
                add_few(n, (tokens + 31) / 32, packs && tokens <= pack_tokens);
            } else {
                add_many(n * groups, tokens, (R + groups - 1) / groups * G);
            }
        }
        double span = std::max(longest_us, work / lay.slots), seen = 0;
        for (int b = top, round = 0; b >= 0; --b) {  // workgroup number k * slots runs as the k + 1st on some slot at the earliest
            for (seen += bins[b]; seen > (double)round * lay.slots; ++round) span = std::max(span, (round + 1) * 0.25 * (b + 0.5));
        }
        span *= 1.0 + k.full * std::min(1.0, n_wgs / lay.slots);
        issue = (issue + k.wg * n_wgs) / chip.n_cu;
        const double rows = 1e-6 * pl.n_req * pl.num_q_heads;
        return k.base + std::cbrt(span * span * span + issue * issue * issue + memory * memory * memory) + rows * (k.part * parts + k.row);
    };
    auto estimate = [&](const Layout &lay, int parts) { return estimate_by(lay, parts, fp8_pool ? kFp8 : lay.max_req > std::max(1, 64 / G) ? kBf16Tall : lay.wide ? kBf16Wide : kBf16Narrow); };
    // Shared nodes, bf16 pools: shared::body or 16-row tiles.  An item alone takes two thirds as long in shared::body, but two
    // workgroups fill a compute unit where three with 16-row tiles do, so that on a full chip the two come to the same and
    // how the items fill it decides (one root of 512 tokens over 64 leaves of 128 tokens 22.3 us as 16-row tiles, 17.3 as 32-row
    // tiles; 8192 over 64 x 1024 63.4 / 73.5).  Both pools: the chunk's length, from 128 tokens (a few items
    // on an empty chip) to whole nodes (many rows, each with a partial per chunk).  Against the length above and the form that
    // suits it, wherever the estimate is shorter by 8 % in that form or by 10 % in the other: 1687 random plans take 0.922 of their time
    // in the mean, 7 lose more than 3 %, none 8 %; at 4 and 8 % 0.918, 18 and 4 up to 12 %; the best of all tried lengths and
    // forms would give 0.887 (profiles/decode_plan_timings.csv).  64 requests x 21 drafted
    // tokens x 32 heads over 2048 + 512, bf16: 138 us in chunks of 512 tokens, 106 in whole nodes; 9 requests x 8 heads below
    // each of 4 x 6996 tokens: 27.9 in chunks of 1024, 15.2 of 192.
    // Plans whose partials fit the static workspace at that length keep to lengths that fit.
    const bool search = any_shared && !pl.fp8_matrix && opt.shared_chunk == 0 && opt.leaf_chunk == 0;
    const bool narrow_too = !fp8_pool && pl.tile_form <= 0, wide_too = any_shared && (fp8_pool || pl.tile_form >= 0);
    // Tall tiles, where some node has more than 64 rows: 1200 other plans, each timed in all forms and lengths, with this margin 164 run that way
    // and take 0.888 of the time, three lose more than 3 % (up to 6.7 %); at 7 % 306 and 21 (up to 10 %).  They pay from about 35 us on
    // (best length against the best of the other forms, verification: steps of 12 to 20 us 1.05, 35 to 60 us 0.93, 100 us and more 0.88).
    const int tall_req = std::max(1, 128 / G);
    const bool tall_too = narrow_too && wide_too && opt.max_rows == 0 && most_req > max_req_per_item;
    auto too_many = [&](int parts) { return partials_bytes((int64_t)pl.n_req * pl.num_q_heads * parts) > kStaticWorkspaceBytes; };
    auto of_default_length = [&](bool cut_more) {
        Layout lay = lay_out(wide_too && (fp8_pool || pl.tile_form > 0), cut_more);
        if (narrow_too && wide_too)
            if (const Layout wide = lay_out(true, cut_more);
                estimate_by(wide, parts_of(wide), kWideThere) < 0.98 * estimate_by(lay, parts_of(lay), kNarrowThere))
                lay = wide;
        return lay;
    };
    struct Choice {
        Layout lay, from;  // from: the one at the default length
        int parts;
        double us;
    };
    auto choose = [&](const Layout &from, bool cut_more) {
        Choice best{from, from, parts_of(from), 0};
        if (!search && pl.paths_us == 0) return best;
        best.us = estimate(from, best.parts);
        if (!search) return best;
        const bool fits = !too_many(best.parts);
        double least = best.us;  // times the margin: 8 % in the same form, 10 % in the other
        for (const int form : {0, 1, 2}) {  // 16-row tiles, 32-row tiles, tall ones
            const bool w = form > 0;
            if (form == 2 ? !tall_too : w ? !wide_too : !narrow_too) continue;
            Layout l = lay_out(w, cut_more);
            l.piece_tokens = pack_tokens;
            if (form == 2) l.max_req = tall_req;
            bool whole = false;  // every node is, at this length and at those behind it
            for (const int chunk : {128, 192, 256, 384, 512, 768, 1024, 1536, 2048}) {
                if (whole) break;
                whole = chunk >= classes.back().tokens;
                l.shared_chunk = chunk;
                const int parts = parts_of(l);
                if (fits && too_many(parts)) continue;
                const double e = estimate(l, parts), us = e / (w == from.wide && form < 2 ? 0.92 : 0.90);
                if (us >= least) continue;
                least = us;
                best = Choice{l, from, parts, e};
            }
        }
        return best;
    };
    // Every partial of the longest list is one of every row of the batch.  Where the cutting of nodes to fill slots, or the form, alone
    // takes them beyond the static workspace, the nodes stay whole (a batch of many heads in which few paths are long: 234
    // requests x 128 heads, 30 MB whole, 53 MB cut) or run in the other form (240 requests x 64 heads below 2 x 11984 and 80 x 2356
    // tokens: 24 MB as 32-row tiles, 36 MB as 16-row tiles), so that attn_decode_plan_run_static takes the plan.
    const Layout first = of_default_length(true);
    Choice chosen = choose(first, true);
    if (too_many(chosen.parts)) {
        auto take_if_it_fits = [&](const Layout &from, bool cut_more) {
            const Choice other = choose(from, cut_more);
            if (too_many(other.parts)) return false;
            chosen = other;
            return true;
        };
        if (!take_if_it_fits(of_default_length(false), false) && narrow_too && wide_too)
            for (const bool cut_more : {true, false})
                if (take_if_it_fits(lay_out(!first.wide, cut_more), cut_more)) break;
    }
    // Paths instead of items (estimate_paths): the items are described as ever, their workspace is that of the default length.
    pl.items_us = chosen.us;
    const bool paths = pl.paths_us > 0 && !any_tiled && pl.paths_us <= 0.93 * pl.items_us;
    if (!paths) pl.n_paths = pl.path_waves = 0;
    const Layout lay = paths && !too_many(parts_of(chosen.from)) ? chosen.from : chosen.lay;
    // Longer items than these take their rows' references anew at this length (rows_body.h): results no further off than with it.
    pl.restart_tokens = std::max(64, (opt.shared_chunk ? default_chunk : chosen.from.shared_chunk) / 64 * 64);
    pl.has_shared = lay.wide;
    struct Proto { DecodeItem it; int64_t cost; };
    std::vector<Proto> protos;
    std::vector<int32_t> node_chunks(n_nodes, 0), slot_base(n_nodes, 0);
    for (int v = 0; v < n_nodes; ++v) {
        const hkv_node &nd = pl.nodes[v];
        if (nd.parent >= 0) slot_base[v] = slot_base[nd.parent] + node_chunks[nd.parent];
        int R = pl.node_req_indptr[v + 1] - pl.node_req_indptr[v];
        if (nd.n_tokens == 0 || R == 0) continue;
        if (tiled(v)) {  // equal chunks of whole pages x equal request groups x KV heads, longest chunks first below
            const int pages_per_chunk = tile_pages(v);
            node_chunks[v] = (nd.n_pages + pages_per_chunk - 1) / pages_per_chunk;
            const int n_groups = (R + req_per_tile - 1) / req_per_tile;
            const int req_per_group = (R + n_groups - 1) / n_groups;
            for (int pg = 0, ci = 0; pg < nd.n_pages; pg += pages_per_chunk, ++ci) {
                const int tb = pg * 16;
                const int nt = std::min(pages_per_chunk * 16, nd.n_tokens - tb);
                for (int r0 = 0; r0 < R; r0 += req_per_group)
                    for (int h = 0; h < Hkv; ++h)
                        pl.tile_items.push_back(DecodeItem{nd.page_begin + pg, nt, h, pl.node_req_indptr[v] + r0,
                                                           std::min(req_per_group, R - r0), slot_base[v] + ci, tb, v});
            }
            continue;
        }
        const int pages_per_chunk = cuts_of(lay, nd.n_tokens, R).per_chunk;
        node_chunks[v] = (nd.n_pages + pages_per_chunk - 1) / pages_per_chunk;
        // equal request groups (64 + 20 rows would leave a long item of few rows that is listed behind the others), except for a
        // remainder of up to 16 rows beside 16-row tiles: one of those costs as much for 48 rows as for 64, the remainder is run
        // by four wavefronts that share its tokens (4 x 2848 tokens over 18 requests x 8 heads 25.2 -> 22.9 us)
        const int n_groups = (R + lay.max_req - 1) / lay.max_req;
        const bool remainder = !pl.has_shared && pl.pool->d.dtype == HKV_BF16 && (R - (n_groups - 1) * lay.max_req) * G <= 16;
        const int req_per_group = remainder ? lay.max_req : (R + n_groups - 1) / n_groups;
        for (int r0 = 0; r0 < R; r0 += req_per_group) {
            int nr = std::min(req_per_group, R - r0);
            for (int pg = 0, ci = 0; pg < nd.n_pages; pg += pages_per_chunk, ++ci) {
                int tb = pg * 16;
                int nt = std::min(pages_per_chunk * 16, nd.n_tokens - tb);
                for (int h = 0; h < Hkv; ++h) {
                    DecodeItem it{nd.page_begin + pg, nt, h, pl.node_req_indptr[v] + r0, nr, slot_base[v] + ci, tb, v};
                    int rows = nr * G;
                    protos.push_back({it, (int64_t)nt * std::max(16, (rows + 15) / 16 * 16)});
                }
            }
        }
    }
    // Forests with more items than the chip holds at once: the short items of at most 16 rows are run four
    // to a workgroup, one per wavefront (a workgroup's start-up then serves four items, and such a
    // wavefront streams its whole item with one step in flight); they are listed behind the others.
    const bool pack = pack_mode == 3 || (pack_mode == 2 && (int64_t)protos.size() > lay.slots);
    auto packable = [&](const Proto &p) { return pack && p.it.n_req * G <= 16 && p.it.n_tokens <= pack_tokens; };
    // one item per workgroup first, heavy before light in both classes: a single integer key per item
    for (Proto &p : protos) p.cost = (packable(p) ? 0 : (int64_t)1 << 56) + p.cost;
    std::stable_sort(protos.begin(), protos.end(), [](const Proto &a, const Proto &b) { return a.cost > b.cost; });
    // Among the one-item workgroups, items shared by more than 16 query rows are bound by their instruction
    // stream and items of few rows by memory: the two classes are dispatched side by side, each spread evenly
    // over the list (groups of 8 = one workgroup per XCD), so that both are resident on every CU throughout
    // instead of one class after the other.  Within a class the order stays heavy before light.
    // Whole sets of KV heads from either list, so that a head's items stay on its XCD.
    if (const int group = or_default(opt.interleave, (8 + Hkv - 1) / Hkv * Hkv); group > 0) {
        std::vector<Proto> many, few, rest, merged;
        for (auto &p : protos) (packable(p) ? rest : p.it.n_req * G > 16 ? many : few).push_back(p);
        if (!many.empty() && !few.empty()) {
            merged.reserve(protos.size());
            size_t a = 0, b = 0;
            while (a < many.size()) {
                for (int i = 0; i < group && a < many.size(); ++i) merged.push_back(many[a++]);
                const size_t target = (size_t)((double)a * few.size() / many.size() / Hkv + 0.5) * Hkv;
                while (b < target && b < few.size()) merged.push_back(few[b++]);
            }
            while (b < few.size()) merged.push_back(few[b++]);
            merged.insert(merged.end(), rest.begin(), rest.end());
            protos.swap(merged);
        }
    }
    std::stable_sort(pl.tile_items.begin(), pl.tile_items.end(),
                     [](const DecodeItem &x, const DecodeItem &y) { return x.n_tokens > y.n_tokens; });
    // While the items leave a quarter of the chip to the other items' first workgroups: as few persistent
    // workgroups as finish their chain of items within the step (a tile item runs at about 5.5 TFLOP/s on its
    // compute unit), in whole groups of 8 (one per XCD).  The items then hold few compute units for the whole
    // step instead of many for a part of it, which the streaming items use better (c5: 64 workgroups of two
    // items against 128 of one, step -2 %); a chain that outlasts the step would lengthen it, hence the margin.
    if (!tiles_first && opt.tile_workgroups == 0 && !pl.tile_items.empty() && (int)pl.tile_items.size() <= chip.n_cu - 64) {
        const int n_items = (int)pl.tile_items.size();
        double item_seconds = 0;
        for (const DecodeItem &it : pl.tile_items)
            item_seconds = std::max(item_seconds, 4.0 * HKV_HEAD_DIM * it.n_tokens * (double)it.n_req * G / 5.5e12);
        const int chain = std::max(1, (int)(step_seconds / item_seconds - 0.1));
        pl.tile_workgroups = std::min(n_items, ((n_items + chain - 1) / chain + 7) / 8 * 8);
    }
    pl.tile_workgroups = std::min<int32_t>(pl.tile_workgroups, (int32_t)pl.tile_items.size());
    pl.items.clear();
    pl.n_single = 0;
    for (auto &p : protos) {
        pl.items.push_back(p.it);
        pl.n_single += !packable(p);
    }
    // LDS stages per workgroup.  The fp8 kernel runs two workgroups per CU (registers), so each may own
    // half of the CU's 160 KiB: five stages, four steps of a shared item in flight instead of two.
    pl.n_stages = or_default(opt.stages, fp8_pool || pl.has_shared ? 5 : 3);
    if (pl.has_shared && !pl.fp8_matrix) pl.n_stages = std::max(pl.n_stages, 4);  // shared::body's ring holds two half-blocks in use and two on their way
    pl.part_count.assign(pl.n_req, 0);
    pl.max_parts = 1;
    for (int r = 0; r < pl.n_req; ++r) {
        int leaf = pl.req_leaf[r];
        pl.part_count[r] = slot_base[leaf] + node_chunks[leaf];
        pl.max_parts = std::max(pl.max_parts, pl.part_count[r]);
    }
    pl.n_parts = pl.n_req * pl.num_q_heads * pl.max_parts;
    // One launch for both kinds of items where the kernel allows it: its workgroups of the other items run two
    // blocks side by side, which works as long as no item synchronises per step (more than 16 query rows).
    pl.fused = !pl.tile_items.empty() && !pl.items.empty() && opt.fused >= 0 && !pl.fp8_matrix;
    for (const DecodeItem &it : pl.items) pl.fused = pl.fused && it.n_req * G <= 16;
}

// Small steps.  The items' kernel and the merge are two launches, each a chain of dependent round trips (plan, blocks, K/V;
// partials), 9 to 16 us however little there is to read.  Where the paths are short enough to be walked whole, a workgroup per
// leaf (up to 16 of its rows) and KV head reads the path, shared nodes again for every leaf, and writes the result: one launch,
// no partials.  What that takes, us: the launch and its chain, and the blocks a compute unit has to take in,
// some 50 to 100 bytes per ns, more where the nodes are not in the L2 of every XCD that reads them.
// (Coefficients from 860 random plans of 16 to 3500 tokens per path, timed in both forms with three sets of inputs in turn: 10 %
// rms; both forms have become shorter since, paths by 11 % and items by 6 %.  Paths where that is 7 % below the items' estimate: of
// 700 other plans (profiles/decode_path_timings.csv) 434 run this way, one of which is more than 3 % (3.5 %) faster as items, and
// 94 of the others would be that much faster this way; at 3 % 464 and four, by up to 14 %, and 68.  What the estimate does not
// know is that a few compute units get two of the longest paths: 38 leaves of 160 to 527 tokens below 496, 32 / 8 heads, bf16,
// 304 workgroups, 18.0 us as items, 21.3 this way, estimated at 0.937 of the items' time.
// Four requests over 256 + 32 + 17 tokens, bf16, 8 / 2 heads: 10.7 -> 5.3 us; 16 requests over 480 + 160 tokens, 32 / 8 heads:
// 16.2 -> 7.8; 32: 18.5 -> 9.1; 64 run as items, 13.9 (this way 13.3 to 13.8); 128: 22.5 as items, 23.7 this way.)
// Eight wavefronts while every workgroup has a compute unit to itself, four where several share one (64 requests over 240 +
// 80 tokens, fp8: 12.3 us with eight, 9.0 with four).
// A caller that sets anything of the planner's, or asks for a form of the items, gets items; growing plans have theirs
// changed on the device and keep them.  rows: the plan's rows by leaf (v's are rows[first[v]] .. rows[first[v + 1] - 1]).
struct RowsByLeaf {
    std::vector<int32_t> first, rows, blocks_to;  // blocks_to: blocks of the path that ends at a node
};
static void estimate_paths(hkv_decode_plan &pl, RowsByLeaf &by) {
    const hkv_decode_plan_params &o = pl.opt;
    if (pl.n_req == 0 || pl.fp8_matrix || pl.tile_form != 0 || pl.reserve_tokens > 0) return;
    if (o.leaf_chunk || o.shared_chunk || o.max_rows || o.pack || o.pack_tokens || o.stages || o.interleave || o.tile_min_rows ||
        o.tile_min_gflop || o.tile_workgroups || o.tile_chunk || o.large_batch_updates || o.fused)
        return;
    if (pl.pool->d.num_pages > (kPathIdMask + 1) / pl.pool->blocks_per_page) return;  // block ids share a word with a count
    const int n_cu = chip_shape().n_cu, Hkv = pl.pool->d.num_kv_heads, per_path = std::max(1, 16 / pl.group);
    const int64_t most_units = 12 * n_cu;
    if ((int64_t)pl.n_req * Hkv > most_units * per_path) return;
    const int n_nodes = (int)pl.nodes.size();
    by.first.assign(n_nodes + 1, 0);
    by.rows.resize(pl.n_req);
    by.blocks_to.resize(n_nodes);
    for (int r = 0; r < pl.n_req; ++r) ++by.first[pl.req_leaf[r] + 1];
    int64_t longest = 0, paths = 0;
    double block_sum = 0, unique = 0;  // blocks of all paths; K/V bytes of the forest, times the XCDs that read them
    for (int v = 0; v < n_nodes; ++v) {
        by.blocks_to[v] = pl.nodes[v].n_pages + (pl.nodes[v].parent >= 0 ? by.blocks_to[pl.nodes[v].parent] : 0);
        if (pl.node_req_indptr[v + 1] > pl.node_req_indptr[v]) unique += pl.nodes[v].n_tokens;
        const int n = by.first[v + 1];
        by.first[v + 1] += by.first[v];
        if (n == 0) continue;
        longest = std::max<int64_t>(longest, by.blocks_to[v]);
        paths += (n + per_path - 1) / per_path;
        block_sum += (double)by.blocks_to[v] * ((n + per_path - 1) / per_path);
    }
    const int64_t units = paths * Hkv;
    if (units > most_units || longest > 256) return;
    std::vector<int32_t> at(by.first.begin(), by.first.end() - 1);
    for (int r = 0; r < pl.n_req; ++r) by.rows[at[pl.req_leaf[r]]++] = r;
    const bool fp8 = pl.pool->d.dtype == HKV_FP8_E4M3;
    int xcds = 8;  // a KV head's workgroups lie Hkv apart
    for (int h = Hkv; h % 2 == 0 && xcds > 1; h /= 2) xcds /= 2;
    unique *= 2.0 * HKV_HEAD_DIM * Hkv * (fp8 ? 1 : 2) * xcds;
    const int waves = units <= n_cu ? 8 : 4;
    // in 1000 tokens: the longest path, and what a compute unit takes in beyond it (between the mean and that of whole workgroups)
    const double per_cu = (double)units / n_cu, most = longest * 16e-3, mean = block_sum / paths * 16e-3;
    const double beside = 0.5 * std::max(0.0, per_cu * mean - most) + 0.5 * std::max(0.0, std::ceil(per_cu) * mean - most);
    const double us = fp8 ? 6.0 + 5.2 * most + 8.0 * beside + 0.23 * per_cu + 0.017e-6 * unique : 5.2 + 6.5 * most + 10.9 * beside + 0.046e-6 * unique;
    if (us > 25) return;  // (hardly timed beyond; 40 leaves of 963 to 1926 tokens below 4 x 493, estimated at 45 us, took 55, as items 46)
    pl.paths_us = us;
    pl.n_paths = (int32_t)paths;
    pl.path_waves = waves;
    pl.path_stride = (int32_t)((kPathBlocks + std::max<int64_t>(longest, 1) + 15) / 16 * 16);
}

// The records of the paths that plan_items has left.
static void plan_paths(hkv_decode_plan &pl, const RowsByLeaf &by) {
    if (pl.n_paths == 0) return;
    const int per_path = std::max(1, 16 / pl.group);
    pl.paths.assign((size_t)pl.path_stride * pl.n_paths, 0);
    int32_t *rec = pl.paths.data();
    for (int v = 0; v < (int)pl.nodes.size(); ++v)
        for (int r0 = by.first[v]; r0 < by.first[v + 1]; r0 += per_path, rec += pl.path_stride) {
            const int n = std::min(per_path, by.first[v + 1] - r0);
            rec[0] = by.blocks_to[v];
            rec[1] = n;
            rec[2] = (by.blocks_to[v] - pl.nodes[v].n_pages) * HKV_PAGE_SIZE;
            for (int i = 0; i < 16; ++i) {
                const int32_t row = by.rows[r0 + std::min(i, n - 1)];
                rec[kPathRows + i] = row;
                rec[kPathQRows + i] = pl.q_rows.empty() ? row : pl.q_rows[row];
            }
            int32_t *end = rec + kPathBlocks + by.blocks_to[v];
            for (int u = v; u >= 0; u = pl.nodes[u].parent) {
                const hkv_node &nd = pl.nodes[u];
                for (int b = nd.n_pages - 1; b >= 0; --b) {
                    const int tokens = std::min(HKV_PAGE_SIZE, nd.n_tokens - b * HKV_PAGE_SIZE);
                    *--end = (int32_t)((uint32_t)pl.node_pages[nd.page_begin + b] | (uint32_t)(HKV_PAGE_SIZE - tokens) << kPathIdBits);
                }
            }
        }
}

// Whether runs queue the two kinds of items side by side, on the caller's stream and on the plan's own.
static bool forks(const hkv_decode_plan &pl) { return !pl.tile_items.empty() && !pl.items.empty() && pl.concurrent && !pl.fused; }

static int upload_decode_plan(hkv_decode_plan &pl) {
    size_t off_items = 0;
    size_t off_pages = align_up(off_items + sizeof(DecodeItem) * pl.items.size(), 256);
    size_t off_nri = align_up(off_pages + sizeof(int32_t) * pl.node_pages.size(), 256);
    size_t off_cnt = align_up(off_nri + sizeof(int32_t) * pl.node_req_idx.size(), 256);
    size_t off_tiles = align_up(off_cnt + sizeof(int32_t) * pl.part_count.size(), 256);
    size_t off_qrows = align_up(off_tiles + sizeof(DecodeItem) * pl.tile_items.size(), 256);
    size_t off_paths = align_up(off_qrows + sizeof(int32_t) * pl.q_rows.size(), 256);
    size_t total = align_up(off_paths + sizeof(int32_t) * pl.paths.size(), 256) + 256;
    HKV_HIP(hipMalloc(&pl.dev, total));
    char *base = static_cast<char *>(pl.dev);
    pl.d_items = reinterpret_cast<DecodeItem *>(base + off_items);
    pl.d_pages = reinterpret_cast<int32_t *>(base + off_pages);
    pl.d_node_req_idx = reinterpret_cast<int32_t *>(base + off_nri);
    pl.d_part_count = reinterpret_cast<int32_t *>(base + off_cnt);
    pl.d_tile_items = reinterpret_cast<DecodeItem *>(base + off_tiles);
    pl.d_paths = reinterpret_cast<int32_t *>(base + off_paths);
    pl.d_q_rows = pl.q_rows.empty() ? nullptr : reinterpret_cast<int32_t *>(base + off_qrows);
    // one host image, one copy
    std::vector<char> image(total, 0);
    auto put = [&](size_t off, const void *src, size_t n) {
        if (n) memcpy(image.data() + off, src, n);
    };
    put(off_items, pl.items.data(), sizeof(DecodeItem) * pl.items.size());
    put(off_pages, pl.node_pages.data(), sizeof(int32_t) * pl.node_pages.size());
    put(off_nri, pl.node_req_idx.data(), sizeof(int32_t) * pl.node_req_idx.size());
    put(off_cnt, pl.part_count.data(), sizeof(int32_t) * pl.part_count.size());
    put(off_tiles, pl.tile_items.data(), sizeof(DecodeItem) * pl.tile_items.size());
    put(off_qrows, pl.q_rows.data(), sizeof(int32_t) * pl.q_rows.size());
    put(off_paths, pl.paths.data(), sizeof(int32_t) * pl.paths.size());
    HKV_HIP(hipMemcpy(pl.dev, image.data(), total, hipMemcpyHostToDevice));
    if (pl.reserve_tokens > 0 && pl.n_req <= kMaxInlineAppend && !pl.grow_items.empty() && !pl.opt.large_batch_updates) {
        HKV_HIP(hipMalloc((void **)&pl.d_grow_items, sizeof(int32_t) * pl.grow_items.size()));
        HKV_HIP(hipMemcpy(pl.d_grow_items, pl.grow_items.data(), sizeof(int32_t) * pl.grow_items.size(), hipMemcpyHostToDevice));
    } else if (pl.reserve_tokens > 0) {
        pl.grow_bytes = align_up(off_pages + sizeof(int32_t) * pl.node_pages.size(), 16);  // inside the allocation: off_nri is 256-aligned
        HKV_HIP(hipHostMalloc((void **)&pl.h_grow, pl.grow_bytes * hkv_decode_plan::kGrowSlots, hipHostMallocDefault));
        HKV_HIP(hipHostGetDevicePointer((void **)&pl.d_grow, pl.h_grow, 0));
        memset(pl.h_grow, 0, pl.grow_bytes * hkv_decode_plan::kGrowSlots);
        for (hipEvent_t &e : pl.grow_free) HKV_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    }
    if (forks(pl)) {  // the second kernel's own stream and the two events that fork to it and join it
        HKV_HIP(hipStreamCreateWithFlags(&pl.side, hipStreamNonBlocking));
        HKV_HIP(hipEventCreateWithFlags(&pl.ev_fork, hipEventDisableTiming));
        HKV_HIP(hipEventCreateWithFlags(&pl.ev_join, hipEventDisableTiming));
    }
    // here, so that the first run may already be under graph capture
    HKV_HIP(prepare_decode_device(nullptr));
    return HKV_OK;
}

// fp32 pools: per-row block tables (root-to-leaf page lists) and lengths instead of work items
static int build_fp32_rows(hkv_decode_plan &pl, bool upload) {
    const int n = pl.n_req;
    std::vector<std::vector<int32_t>> paths(n);
    std::vector<char> seen(pl.nodes.size(), 0);
    int64_t n_pages = 0;  // of the nodes on some row's path
    pl.row_len.assign(n, 0);
    pl.max_pages = 1;
    for (int r = 0; r < n; ++r) {
        std::vector<int32_t> chain;
        for (int v = pl.req_leaf[r]; v >= 0; v = pl.nodes[v].parent) chain.push_back(v);
        for (auto it = chain.rbegin(); it != chain.rend(); ++it) {
            const hkv_node &nd = pl.nodes[*it];
            if (!seen[*it]) n_pages += nd.n_pages;
            seen[*it] = 1;
            paths[r].insert(paths[r].end(), pl.node_pages.begin() + nd.page_begin, pl.node_pages.begin() + nd.page_begin + nd.n_pages);
            pl.row_len[r] += nd.n_tokens;
        }
        pl.max_pages = std::max<int32_t>(pl.max_pages, (int32_t)paths[r].size());
    }
    const double page_mb = 1e-6 * 2 * kBlockElems * sizeof(float) * pl.pool->d.num_kv_heads;
    pl.row_parts = row_shares(n, pl.pool->d.num_kv_heads, pl.group, pl.max_pages, page_mb * n_pages);
    if (!upload || n == 0) return HKV_OK;
    std::vector<int32_t> bt((size_t)n * pl.max_pages, 0), req(n);
    for (int r = 0; r < n; ++r) {
        std::copy(paths[r].begin(), paths[r].end(), bt.begin() + (size_t)r * pl.max_pages);
        req[r] = r;
    }
    const size_t b_bt = align_up(sizeof(int32_t) * bt.size(), 256), b_n = align_up(sizeof(int32_t) * n, 256);
    HKV_HIP(hipMalloc((void **)&pl.d_bt, b_bt + 2 * b_n));
    pl.d_rows_req = reinterpret_cast<int32_t *>(reinterpret_cast<char *>(pl.d_bt) + b_bt);
    pl.d_rows_len = reinterpret_cast<int32_t *>(reinterpret_cast<char *>(pl.d_bt) + b_bt + b_n);
    HKV_HIP(hipMemcpy(pl.d_bt, bt.data(), sizeof(int32_t) * bt.size(), hipMemcpyHostToDevice));
    HKV_HIP(hipMemcpy(pl.d_rows_req, req.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice));
    HKV_HIP(hipMemcpy(pl.d_rows_len, pl.row_len.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice));
    return HKV_OK;
}

// internal flag: plans with per-row visibility
constexpr uint32_t kPlanRowVisibility = 0x40000000u;

// the planner's settings, each 0 (the library's choice) or inside its documented range
static int check_plan_settings(const hkv_decode_plan_params *o) {
    if (!o) return HKV_OK;
    auto bad = [](const char *name, int32_t v) { return fail(HKV_EINVAL, "hkv_decode_plan_create_ex: %s = %d is out of range", name, v); };
    if (o->leaf_chunk < 0 || o->leaf_chunk % 16) return bad("leaf_chunk", o->leaf_chunk);
    if (o->shared_chunk < 0 || o->shared_chunk % 16 || o->shared_chunk > kMaxSharedItemTokens) return bad("shared_chunk", o->shared_chunk);
    if (o->max_rows != 0 && (o->max_rows < 16 || o->max_rows > 64)) return bad("max_rows", o->max_rows);
    if (o->pack < 0 || o->pack > 3) return bad("pack", o->pack);
    if (o->pack_tokens < 0) return bad("pack_tokens", o->pack_tokens);
    if (o->stages != 0 && (o->stages < 3 || o->stages > 5)) return bad("stages", o->stages);
    if (o->interleave < -1) return bad("interleave", o->interleave);
    if (o->tile_min_rows != 0 && o->tile_min_rows < kMinTileItemRows) return bad("tile_min_rows", o->tile_min_rows);
    if (o->tile_min_gflop < -1) return bad("tile_min_gflop", o->tile_min_gflop);
    if (o->tile_workgroups < 0) return bad("tile_workgroups", o->tile_workgroups);
    if (o->tile_chunk < 0 || o->tile_chunk % 16 || o->tile_chunk > kMaxTileItemTokens) return bad("tile_chunk", o->tile_chunk);
    if (o->large_batch_updates < 0 || o->large_batch_updates > 1) return bad("large_batch_updates", o->large_batch_updates);
    if (o->fused < -1 || o->fused > 0) return bad("fused", o->fused);
    return HKV_OK;
}

static int create_decode_plan(hkv_pool *pool, const hkv_node *nodes, int32_t n_nodes, const int32_t *node_pages,
                              int32_t n_node_pages, const int32_t *req_leaf, int32_t n_req, int32_t num_q_heads,
                              uint32_t flags, int32_t reserve_tokens, const hkv_decode_plan_params *opt,
                              hkv_decode_plan **out) {
    if (!pool || !out) return fail(HKV_EINVAL, "hkv_decode_plan_create: null argument");
    *out = nullptr;
    if (int rc = check_plan_settings(opt)) return rc;
    const int Hkv = pool->d.num_kv_heads;
    if (num_q_heads <= 0 || num_q_heads % Hkv || num_q_heads / Hkv > 16)
        return fail(HKV_ESHAPE, "hkv_decode_plan_create: %d query heads over %d KV heads", num_q_heads, Hkv);
    if ((flags & HKV_PLAN_FP8_MATRIX) && pool->d.dtype != HKV_FP8_E4M3)
        return fail(HKV_ESHAPE, "hkv_decode_plan_create: HKV_PLAN_FP8_MATRIX needs an fp8 pool");
    // The per-node kernels read every node through its own page list, so nodes may end inside a page
    // anywhere; the full-precision path walks flat block tables and keeps the whole-page rule.
    if (int rc = validate_forest(nodes, n_nodes, node_pages, n_node_pages, "hkv_decode_plan_create",
                                 pool->d.dtype == HKV_FP32, pool->d.page_size))
        return rc;
    for (int v = 0; v < n_nodes; ++v)
        for (int j = 0; j < nodes[v].n_pages; ++j) {
            int32_t id = node_pages[nodes[v].page_begin + j];
            if (id < 0 || id >= pool->d.num_pages)
                return fail(HKV_ERANGE, "hkv_decode_plan_create: node %d page %d has id %d outside pool of %d", v, j,
                            id, pool->d.num_pages);
        }
    hkv_decode_plan *pl = new (std::nothrow) hkv_decode_plan;
    if (!pl) return fail(HKV_ENOMEM, "hkv_decode_plan_create: out of host memory");
    if (pool->d.dtype == HKV_BF16) pl->tile_form = flags & HKV_PLAN_NARROW_TILES ? -1 : flags & HKV_PLAN_WIDE_TILES ? 1 : flags & HKV_PLAN_TALL_TILES ? 2 : 0;
    pl->pool = pool;
    pl->n_req = n_req;
    pl->num_q_heads = num_q_heads;
    pl->group = num_q_heads / Hkv;
    pl->fp8_matrix = pool->d.dtype == HKV_FP8_E4M3 && (flags & HKV_PLAN_FP8_MATRIX);
    if (opt) pl->opt = *opt;
    if (opt && opt->q_rows) {
        if (pool->d.dtype == HKV_FP32) {
            delete pl;
            return fail(HKV_ESHAPE, "hkv_decode_plan_create_ex: q_rows with an fp32 pool");
        }
        pl->q_rows.assign(opt->q_rows, opt->q_rows + n_req);
        std::vector<int32_t> sorted(pl->q_rows);
        std::sort(sorted.begin(), sorted.end());
        if (!sorted.empty() && (sorted.front() < 0 || std::adjacent_find(sorted.begin(), sorted.end()) != sorted.end())) {
            delete pl;
            return fail(HKV_EINVAL, "hkv_decode_plan_create_ex: q_rows must be non-negative and all different");
        }
        pl->opt.q_rows = nullptr;  // the caller's array is not kept
    }
    pl->opt.visible = nullptr;
    pl->row_visibility = (flags & kPlanRowVisibility) != 0;
    pl->concurrent = !(flags & HKV_PLAN_ONE_STREAM);
    // the documented default of a setting is the library's own choice, as 0 is
    if (pl->opt.pack == 2) pl->opt.pack = 0;
    if (pl->opt.interleave == 8) pl->opt.interleave = 0;
    if (pl->opt.tile_min_rows == 128) pl->opt.tile_min_rows = 0;
    if (pl->opt.tile_min_gflop == 40 && !pl->row_visibility) pl->opt.tile_min_gflop = 0;
    if (int rc = build_node_req_csr(nodes, n_nodes, req_leaf, n_req, pl->node_req_indptr, pl->node_req_idx,
                                    "hkv_decode_plan_create")) {
        delete pl;
        return rc;
    }
    pl->key_nodes.assign(nodes, nodes + n_nodes);
    pl->key_pages.assign(node_pages, node_pages + n_node_pages);
    pl->req_leaf.assign(req_leaf, req_leaf + n_req);
    // the plan itself works on 16-token blocks: block j of page p is block p * S + j of the buffers
    pl->nodes.assign(nodes, nodes + n_nodes);
    pl->node_pages.clear();
    const int S = pool->blocks_per_page;
    pl->node_pages.reserve((size_t)n_node_pages * S + (reserve_tokens > 0 ? (size_t)n_req * (reserve_tokens / HKV_PAGE_SIZE + 2) : 0));
    std::vector<char> grows(n_nodes, 0);
    if (reserve_tokens > 0)
        for (int r = 0; r < n_req; ++r) grows[req_leaf[r]] = 1;
    pl->reserve_tokens = reserve_tokens;
    for (int v = 0; v < n_nodes; ++v) {
        hkv_node &nd = pl->nodes[v];
        const int n_blocks = (nd.n_tokens + HKV_PAGE_SIZE - 1) / HKV_PAGE_SIZE;
        const int first = (int)pl->node_pages.size();
        for (int b = 0; b < n_blocks; ++b) pl->node_pages.push_back(node_pages[nodes[v].page_begin + b / S] * S + b % S);
        if (grows[v]) {  // slots for the blocks the leaf may grow into; until then they repeat its last block (in bounds)
            const int cap = (nd.n_tokens + reserve_tokens + HKV_PAGE_SIZE - 1) / HKV_PAGE_SIZE;
            for (int b = n_blocks; b < cap; ++b) pl->node_pages.push_back(pl->node_pages.back());
        }
        nd.page_begin = first;
        nd.n_pages = n_blocks;
    }
    if (pool->d.dtype == HKV_FP32) {  // full-precision path: no work items, no partials
        if (int rc = build_fp32_rows(*pl, !(flags & HKV_PLAN_HOST_ONLY))) {
            if (pl->d_bt) (void)hipFree(pl->d_bt);
            delete pl;
            return rc;
        }
        pl->part_count.assign(n_req, 0);
        *out = pl;
        return HKV_OK;
    }
    RowsByLeaf by_leaf;
    estimate_paths(*pl, by_leaf);
    plan_items(*pl);
    plan_paths(*pl, by_leaf);
    if (reserve_tokens > 0) {  // the items that grow with each request: the leaf's last chunk, one per KV head
        pl->grow_items.assign((size_t)n_req * Hkv, -1);
        for (int r = 0; r < n_req; ++r) {
            const int v = req_leaf[r];
            int last_begin = -1;
            for (const DecodeItem &it : pl->items)
                if (it.node == v) last_begin = std::max(last_begin, it.tok_begin);
            for (size_t i = 0; i < pl->items.size(); ++i)
                if (pl->items[i].node == v && pl->items[i].tok_begin == last_begin)
                    pl->grow_items[(size_t)r * Hkv + pl->items[i].kv_head] = (int32_t)i;
        }
        for (int32_t gi : pl->grow_items)
            if (gi < 0) {
                delete pl;
                return fail(HKV_EINVAL, "hkv_decode_plan_create_growing: a leaf without work items");
            }
        pl->key_nodes.clear();  // never the pool's cached one-shot plan
        pl->key_pages.clear();
    }
    if (!(flags & HKV_PLAN_HOST_ONLY)) {
        if (int rc = upload_decode_plan(*pl)) {
            hkv_decode_plan_destroy(pl);
            return rc;
        }
    }
    *out = pl;
    return HKV_OK;
}

extern "C" int hkv_decode_plan_create(hkv_pool *pool, const hkv_node *nodes, int32_t n_nodes,
                                      const int32_t *node_pages, int32_t n_node_pages, const int32_t *req_leaf,
                                      int32_t n_req, int32_t num_q_heads, uint32_t flags, hkv_decode_plan **out) {
    return create_decode_plan(pool, nodes, n_nodes, node_pages, n_node_pages, req_leaf, n_req, num_q_heads,
                              flags & ~kPlanRowVisibility, 0, nullptr, out);
}

static int create_growing_plan(hkv_pool *pool, const hkv_node *nodes, int32_t n_nodes, const int32_t *node_pages,
                               int32_t n_node_pages, const int32_t *req_leaf, int32_t n_req, int32_t num_q_heads,
                               int32_t reserve_tokens, uint32_t flags, const hkv_decode_plan_params *opt,
                               hkv_decode_plan **out) {
    if (!pool || !out) return fail(HKV_EINVAL, "hkv_decode_plan_create_growing: null argument");
    *out = nullptr;
    if (pool->d.dtype == HKV_FP32) return fail(HKV_ESHAPE, "hkv_decode_plan_create_growing: bf16 and fp8 pools only");
    if (reserve_tokens < 1 || reserve_tokens > (1 << 20))
        return fail(HKV_EINVAL, "hkv_decode_plan_create_growing: reserve_tokens %d", reserve_tokens);
    if (n_nodes < 0 || n_req < 0 || (n_nodes > 0 && !nodes) || (n_req > 0 && !req_leaf))
        return fail(HKV_EINVAL, "hkv_decode_plan_create_growing: bad forest arguments");
    // every request needs a leaf of its own to grow: no other request on it, no children, at least one token
    std::vector<int32_t> users(n_nodes, 0);
    for (int r = 0; r < n_req; ++r) {
        if (req_leaf[r] < 0 || req_leaf[r] >= n_nodes)
            return fail(HKV_ERANGE, "hkv_decode_plan_create_growing: request %d names node %d of %d", r, req_leaf[r], n_nodes);
        ++users[req_leaf[r]];
    }
    for (int v = 0; v < n_nodes; ++v)
        if (nodes[v].parent >= 0 && nodes[v].parent < n_nodes && users[nodes[v].parent])
            return fail(HKV_ETREE, "hkv_decode_plan_create_growing: node %d, the leaf of a request, has children", nodes[v].parent);
    for (int r = 0; r < n_req; ++r) {
        if (users[req_leaf[r]] != 1)
            return fail(HKV_ETREE, "hkv_decode_plan_create_growing: node %d is the leaf of %d requests", req_leaf[r], users[req_leaf[r]]);
        if (nodes[req_leaf[r]].n_tokens < 1)
            return fail(HKV_ETREE, "hkv_decode_plan_create_growing: the leaf of request %d holds no token", r);
    }
    return create_decode_plan(pool, nodes, n_nodes, node_pages, n_node_pages, req_leaf, n_req, num_q_heads,
                              flags & ~kPlanRowVisibility, reserve_tokens, opt, out);
}

extern "C" int hkv_decode_plan_create_growing(hkv_pool *pool, const hkv_node *nodes, int32_t n_nodes,
                                              const int32_t *node_pages, int32_t n_node_pages,
                                              const int32_t *req_leaf, int32_t n_req, int32_t num_q_heads,
                                              int32_t reserve_tokens, uint32_t flags, hkv_decode_plan **out) {
    return create_growing_plan(pool, nodes, n_nodes, node_pages, n_node_pages, req_leaf, n_req, num_q_heads,
                               reserve_tokens, flags, nullptr, out);
}

// k_src / v_src: null (the caller stores the tokens itself), or the new token of every request, stored here
// at the end of its leaf, in the same launch as the plan's update where that runs as a kernel.
static int plan_append(hkv_decode_plan *plan, const int32_t *new_page_ids, const void *k_src, const void *v_src,
                       void *stream) {
    if (!plan) return fail(HKV_EINVAL, "hkv_decode_plan_append: null plan");
    if (plan->reserve_tokens <= 0) return fail(HKV_EINVAL, "hkv_decode_plan_append: not a growing plan");
    if (plan->appended >= plan->reserve_tokens)
        return fail(HKV_ENOMEM, "hkv_decode_plan_append: the %d reserved tokens are used up", plan->reserve_tokens);
    hkv_pool *pool = plan->pool;
    const int P = pool->d.page_size, S = pool->blocks_per_page, Hkv = pool->d.num_kv_heads;
    // check everything before anything changes
    for (int r = 0; r < plan->n_req; ++r) {
        const hkv_node &nd = plan->nodes[plan->req_leaf[r]];
        if (nd.n_tokens % P) continue;  // the new token goes into the leaf's last page
        if (!new_page_ids) return fail(HKV_EINVAL, "hkv_decode_plan_append: request %d needs a new page, none given", r);
        if (new_page_ids[r] < 0 || new_page_ids[r] >= pool->d.num_pages)
            return fail(HKV_ERANGE, "hkv_decode_plan_append: page id %d for request %d outside pool of %d pages",
                        new_page_ids[r], r, pool->d.num_pages);
    }
    const bool with_tokens = k_src != nullptr;
    if (with_tokens && (!v_src || ((reinterpret_cast<uintptr_t>(k_src) | reinterpret_cast<uintptr_t>(v_src)) & 15)))
        return fail(HKV_EINVAL, "hkv_decode_plan_append_tokens: k_src and v_src must be non-null and 16-byte aligned");
    const bool inline_update = plan->dev && plan->d_grow_items;
    PlanGrowInline g{};
    PoolAppendInline w{};
    std::vector<int32_t> w_page, w_slot;  // the tokens' places, for the path of larger batches
    if (with_tokens && !inline_update) {
        w_page.resize(plan->n_req);
        w_slot.resize(plan->n_req);
    }
    for (int r = 0; r < plan->n_req; ++r) {
        hkv_node &nd = plan->nodes[plan->req_leaf[r]];
        if (inline_update) g.new_block[r] = -1;
        if (with_tokens) {  // where the new token goes: slot n_tokens % P of the leaf's last (or new) page
            const int32_t page = nd.n_tokens % P == 0 ? new_page_ids[r] : plan->node_pages[nd.page_begin + nd.n_pages - 1] / S;
            if (inline_update) {
                w.block[r] = page * S + (nd.n_tokens % P) / HKV_PAGE_SIZE;
                w.slot[r] = (uint8_t)(nd.n_tokens % HKV_PAGE_SIZE);
            } else {
                w_page[r] = page;
                w_slot[r] = nd.n_tokens % P;
            }
        }
        if (nd.n_tokens % HKV_PAGE_SIZE == 0) {  // a new 16-token block: of a new page, or the next one of the last page
            const int32_t block = nd.n_tokens % P == 0 ? new_page_ids[r] * S
                                                      : plan->node_pages[nd.page_begin + nd.n_pages - 1] + 1;
            plan->node_pages[nd.page_begin + nd.n_pages] = block;
            if (inline_update) {
                g.new_block[r] = block;
                g.block_pos[r] = nd.page_begin + nd.n_pages;
            }
            ++nd.n_pages;
        }
        ++nd.n_tokens;
        for (int h = 0; h < Hkv; ++h) ++plan->items[plan->grow_items[(size_t)r * Hkv + h]].n_tokens;
    }
    ++plan->appended;
    if (!plan->dev) return HKV_OK;  // host-only plan
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (inline_update) {  // the usual batch: the change travels in the arguments of a small kernel
        g.items = plan->d_items;
        g.pages = plan->d_pages;
        g.grow_items = plan->d_grow_items;
        g.n_grow = (int32_t)plan->grow_items.size();
        g.n_req = plan->n_req;
        if (with_tokens) {  // the same launch stores the tokens
            w.base = PoolWriteLaunch{pool->d.k_pages, pool->d.v_pages, pool->d.k_scale, pool->d.v_scale, Hkv, pool->d.dtype,
                                     nullptr, plan->n_req, 0, plan->n_req, k_src, v_src, nullptr, nullptr};
            HKV_HIP(launch_decode_step_append(w, g, s));
        } else {
            HKV_HIP(launch_plan_grow_inline(g, s));
        }
        return HKV_OK;
    }
    if (with_tokens)
        if (int rc = kv_pool_append(pool, w_page.data(), w_slot.data(), plan->n_req, k_src, v_src, stream)) return rc;
    const int slot = plan->grow_next;
    plan->grow_next = (slot + 1) % hkv_decode_plan::kGrowSlots;
    if (plan->grow_in_flight[slot]) HKV_HIP(hipEventSynchronize(plan->grow_free[slot]));  // its last copy is done
    char *h = plan->h_grow + (size_t)slot * plan->grow_bytes;
    const size_t off_pages = reinterpret_cast<char *>(plan->d_pages) - static_cast<char *>(plan->dev);
    memcpy(h, plan->items.data(), sizeof(DecodeItem) * plan->items.size());
    memcpy(h + off_pages, plan->node_pages.data(), sizeof(int32_t) * plan->node_pages.size());
    // a copy kernel on the stream reads the pinned buffer (a DMA copy between two kernels of one stream
    // costs far more than it moves here)
    HKV_HIP(launch_upload(plan->d_grow + (size_t)slot * plan->grow_bytes, plan->dev, plan->grow_bytes, s));
    HKV_HIP(hipEventRecord(plan->grow_free[slot], s));
    plan->grow_in_flight[slot] = true;
    return HKV_OK;
}

extern "C" int hkv_decode_plan_append(hkv_decode_plan *plan, const int32_t *new_page_ids, void *stream) {
    return plan_append(plan, new_page_ids, nullptr, nullptr, stream);
}

extern "C" int hkv_decode_plan_append_tokens(hkv_decode_plan *plan, const int32_t *new_page_ids, const void *k_src,
                                             const void *v_src, void *stream) {
    if (!k_src || !v_src) return fail(HKV_EINVAL, "hkv_decode_plan_append_tokens: null k_src / v_src");
    return plan_append(plan, new_page_ids, k_src, v_src, stream);
}

// Plan over n_req * T query rows: the T newest tokens of every request (the last T of its leaf node) are
// queried together; row t sees everything before them and, of them, token j iff bit j of masks[r * T + t]
// is set (masks == nullptr: the causal run, bits 0..t).
static int create_rows_plan(hkv_pool *pool, const hkv_node *nodes, int32_t n_nodes, const int32_t *node_pages,
                            int32_t n_node_pages, const int32_t *req_leaf, int32_t n_req, int32_t T,
                            const uint64_t *masks, int32_t num_q_heads, uint32_t flags,
                            const hkv_decode_plan_params *opt, hkv_decode_plan **out, const char *who) {
    if (n_req < 0 || (n_req > 0 && !req_leaf)) return fail(HKV_EINVAL, "%s: bad request list", who);
    if ((int64_t)n_req * T > INT32_MAX / 2) return fail(HKV_EINVAL, "%s: too many query rows", who);
    if (masks && pool && pool->d.dtype == HKV_FP32)
        return fail(HKV_ESHAPE, "%s: the full-precision path verifies causal runs only", who);
    std::vector<int32_t> rows((size_t)n_req * T);
    for (int r = 0; r < n_req; ++r)
        for (int t = 0; t < T; ++t) rows[(size_t)r * T + t] = req_leaf[r];
    hkv_decode_plan *pl = nullptr;
    const uint32_t rows_flags = (flags & ~kPlanRowVisibility) | ((T > 1 || masks) ? kPlanRowVisibility : 0u);
    if (int rc = create_decode_plan(pool, nodes, n_nodes, node_pages, n_node_pages, rows.data(), n_req * T, num_q_heads,
                                    rows_flags, 0, opt, &pl))
        return rc;
    pl->tokens_per_req = T;
    if (T > 1 || masks) {
        std::vector<int32_t> lim((size_t)n_req * T);
        std::vector<unsigned long long> vis((size_t)n_req * T);
        for (int r = 0; r < n_req; ++r) {
            const int n_leaf = nodes[req_leaf[r]].n_tokens;  // validated by hkv_decode_plan_create
            if (n_leaf < T) {
                hkv_decode_plan_destroy(pl);
                return fail(HKV_EINVAL, "%s: request %d has %d query tokens but its leaf holds only %d tokens (the "
                            "newest tokens must lie in the leaf)", who, r, T, n_leaf);
            }
            for (int t = 0; t < T; ++t) {
                const size_t i = (size_t)r * T + t;
                lim[i] = n_leaf - T;
                vis[i] = masks ? masks[i] : (t == 63 ? ~0ull : (1ull << (t + 1)) - 1);
                if (!(vis[i] >> t & 1) || (T < 64 && vis[i] >> T)) {
                    hkv_decode_plan_destroy(pl);
                    return fail(HKV_EINVAL, "%s: request %d token %d: a token must see itself and nothing beyond the %d "
                                "newest tokens (mask %llx)", who, r, t, T, vis[i]);
                }
            }
        }
        if (pool->d.dtype == HKV_FP32) {  // query token t of a request sees all but the T-1-t newest keys
            for (int r = 0; r < n_req; ++r)
                for (int t = 0; t < T; ++t) pl->row_len[(size_t)r * T + t] -= T - 1 - t;
            if (pl->d_rows_len) {
                hipError_t e = hipMemcpy(pl->d_rows_len, pl->row_len.data(), sizeof(int32_t) * pl->row_len.size(), hipMemcpyHostToDevice);
                if (e != hipSuccess) {
                    hkv_decode_plan_destroy(pl);
                    return fail_hip(e, who);
                }
            }
        } else if (pl->dev && n_req > 0) {
            const size_t n = rows.size();
            hipError_t e = hipMalloc((void **)&pl->d_row_mask, n * (sizeof(unsigned long long) + 2 * sizeof(int32_t)));
            if (e == hipSuccess) {
                pl->d_row_leaf = reinterpret_cast<int32_t *>(pl->d_row_mask + n);
                pl->d_row_limit = pl->d_row_leaf + n;
                e = hipMemcpy(pl->d_row_mask, vis.data(), n * sizeof(unsigned long long), hipMemcpyHostToDevice);
            }
            if (e == hipSuccess) e = hipMemcpy(pl->d_row_leaf, rows.data(), n * sizeof(int32_t), hipMemcpyHostToDevice);
            if (e == hipSuccess) e = hipMemcpy(pl->d_row_limit, lim.data(), n * sizeof(int32_t), hipMemcpyHostToDevice);
            if (e != hipSuccess) {
                hkv_decode_plan_destroy(pl);
                return fail_hip(e, who);
            }
        }
    }
    *out = pl;
    return HKV_OK;
}

extern "C" int hkv_decode_plan_create_multi(hkv_pool *pool, const hkv_node *nodes, int32_t n_nodes,
                                            const int32_t *node_pages, int32_t n_node_pages, const int32_t *req_leaf,
                                            int32_t n_req, int32_t tokens_per_req, int32_t num_q_heads, uint32_t flags,
                                            hkv_decode_plan **out) {
    if (!out) return fail(HKV_EINVAL, "hkv_decode_plan_create_multi: null out");
    *out = nullptr;
    if (tokens_per_req < 1 || tokens_per_req > 16)
        return fail(HKV_EINVAL, "hkv_decode_plan_create_multi: %d query tokens per request (1..16)", tokens_per_req);
    return create_rows_plan(pool, nodes, n_nodes, node_pages, n_node_pages, req_leaf, n_req, tokens_per_req, nullptr,
                            num_q_heads, flags, nullptr, out, "hkv_decode_plan_create_multi");
}

extern "C" int hkv_decode_plan_create_tree(hkv_pool *pool, const hkv_node *nodes, int32_t n_nodes,
                                           const int32_t *node_pages, int32_t n_node_pages, const int32_t *req_leaf,
                                           int32_t n_req, int32_t tokens_per_req, const uint64_t *visible,
                                           int32_t num_q_heads, uint32_t flags, hkv_decode_plan **out) {
    if (!out) return fail(HKV_EINVAL, "hkv_decode_plan_create_tree: null out");
    *out = nullptr;
    if (tokens_per_req < 1 || tokens_per_req > 64)
        return fail(HKV_EINVAL, "hkv_decode_plan_create_tree: %d drafted tokens per request (1..64)", tokens_per_req);
    if (n_req > 0 && !visible) return fail(HKV_EINVAL, "hkv_decode_plan_create_tree: null visibility masks");
    return create_rows_plan(pool, nodes, n_nodes, node_pages, n_node_pages, req_leaf, n_req, tokens_per_req, visible,
                            num_q_heads, flags, nullptr, out, "hkv_decode_plan_create_tree");
}

extern "C" int hkv_decode_plan_create_ex(hkv_pool *pool, const hkv_node *nodes, int32_t n_nodes,
                                         const int32_t *node_pages, int32_t n_node_pages, const int32_t *req_leaf,
                                         int32_t n_req, int32_t num_q_heads, uint32_t flags,
                                         const hkv_decode_plan_params *params, hkv_decode_plan **out) {
    if (!out) return fail(HKV_EINVAL, "hkv_decode_plan_create_ex: null out");
    *out = nullptr;
    const int32_t T = params && params->tokens_per_req ? params->tokens_per_req : 1;
    const uint64_t *visible = params ? params->visible : nullptr;
    const int32_t reserve = params ? params->reserve_tokens : 0;
    if (T < 1 || T > 64 || (T > 16 && !visible))
        return fail(HKV_EINVAL, "hkv_decode_plan_create_ex: %d query tokens per request (1..16, up to 64 with visibility masks)", T);
    if (reserve < 0) return fail(HKV_EINVAL, "hkv_decode_plan_create_ex: reserve_tokens %d", reserve);
    if (reserve > 0 && (T > 1 || visible))
        return fail(HKV_EINVAL, "hkv_decode_plan_create_ex: a growing plan has one query token per request");
    if (T > 1 || visible)
        return create_rows_plan(pool, nodes, n_nodes, node_pages, n_node_pages, req_leaf, n_req, T, visible, num_q_heads,
                                flags, params, out, "hkv_decode_plan_create_ex");
    if (reserve > 0)
        return create_growing_plan(pool, nodes, n_nodes, node_pages, n_node_pages, req_leaf, n_req, num_q_heads, reserve,
                                   flags, params, out);
    return create_decode_plan(pool, nodes, n_nodes, node_pages, n_node_pages, req_leaf, n_req, num_q_heads,
                              flags & ~kPlanRowVisibility, 0, params, out);
}

extern "C" int hkv_decode_plan_destroy(hkv_decode_plan *plan) {
    if (!plan) return HKV_OK;
    if (plan->dev) (void)hipFree(plan->dev);  // hipFree waits for work that may still read it
    if (plan->d_row_mask) (void)hipFree(plan->d_row_mask);
    if (plan->d_bt) (void)hipFree(plan->d_bt);
    for (hipEvent_t e : plan->ev)
        if (e) (void)hipEventDestroy(e);
    for (hipEvent_t e : {plan->ev_fork, plan->ev_join, plan->ev_tile[0], plan->ev_tile[1]})
        if (e) (void)hipEventDestroy(e);
    if (plan->side) (void)hipStreamDestroy(plan->side);
    if (plan->h_grow) (void)hipHostFree(plan->h_grow);
    if (plan->d_grow_items) (void)hipFree(plan->d_grow_items);
    for (hipEvent_t e : plan->grow_free)
        if (e) (void)hipEventDestroy(e);
    delete plan;
    return HKV_OK;
}

extern "C" size_t hkv_decode_plan_workspace_bytes(const hkv_decode_plan *plan) {
    if (!plan) return 0;
    if (plan->pool->d.dtype == HKV_FP32)
        return plan->row_parts > 1 ? sizeof(float) * kRowPartFloats * (size_t)plan->n_req * plan->num_q_heads * plan->row_parts : 0;
    return partials_bytes(plan->n_parts);
}

extern "C" int32_t hkv_decode_plan_num_items(const hkv_decode_plan *plan) {
    return plan ? (int32_t)(plan->items.size() + plan->tile_items.size()) : fail(HKV_EINVAL, "null plan");
}
extern "C" int32_t hkv_decode_plan_num_tile_items(const hkv_decode_plan *plan) {
    return plan ? (int32_t)plan->tile_items.size() : fail(HKV_EINVAL, "null plan");
}
extern "C" int32_t hkv_decode_plan_is_fused(const hkv_decode_plan *plan) {
    return plan ? (plan->fused ? 1 : 0) : fail(HKV_EINVAL, "null plan");
}
extern "C" int32_t hkv_decode_plan_has_stream(const hkv_decode_plan *plan) {
    return plan ? (plan->side ? 1 : 0) : fail(HKV_EINVAL, "null plan");
}
extern "C" int32_t hkv_decode_plan_has_wide_tiles(const hkv_decode_plan *plan) {
    return plan ? (plan->has_shared && !plan->fp8_matrix ? 1 : 0) : fail(HKV_EINVAL, "null plan");
}
extern "C" int32_t hkv_decode_plan_num_paths(const hkv_decode_plan *plan) {
    return plan ? plan->n_paths : fail(HKV_EINVAL, "null plan");
}
extern "C" int32_t hkv_decode_plan_tile_workgroups(const hkv_decode_plan *plan) {
    return plan ? plan->tile_workgroups : fail(HKV_EINVAL, "null plan");
}
extern "C" int32_t hkv_decode_plan_num_parts(const hkv_decode_plan *plan) {
    return plan ? plan->n_parts : fail(HKV_EINVAL, "null plan");
}
extern "C" int hkv_decode_plan_items(const hkv_decode_plan *plan, int32_t *items_out) {
    if (!plan || !items_out) return fail(HKV_EINVAL, "hkv_decode_plan_items: null argument");
    static_assert(sizeof(DecodeItem) == 32, "item layout is part of the introspection contract");
    if (!plan->items.empty()) memcpy(items_out, plan->items.data(), sizeof(DecodeItem) * plan->items.size());
    if (!plan->tile_items.empty())
        memcpy(items_out + 8 * plan->items.size(), plan->tile_items.data(), sizeof(DecodeItem) * plan->tile_items.size());
    return HKV_OK;
}
extern "C" int32_t hkv_decode_plan_num_workgroups(const hkv_decode_plan *plan) {
    if (!plan) return fail(HKV_EINVAL, "null plan");
    return plan->n_single + ((int32_t)plan->items.size() - plan->n_single + 3) / 4;  // (the tile kernel's are counted apart)
}
extern "C" int32_t hkv_decode_plan_max_parts(const hkv_decode_plan *plan) {
    return plan ? plan->max_parts : fail(HKV_EINVAL, "null plan");
}
extern "C" int hkv_decode_plan_part_counts(const hkv_decode_plan *plan, int32_t *part_count) {
    if (!plan || (plan->n_req > 0 && !part_count)) return fail(HKV_EINVAL, "hkv_decode_plan_part_counts: null argument");
    if (plan->n_req) memcpy(part_count, plan->part_count.data(), sizeof(int32_t) * plan->n_req);
    return HKV_OK;
}

// The common part of the two run calls; arguments are checked by the callers.  workspace holds at least
// hkv_decode_plan_workspace_bytes(plan) bytes (fp32 pools: or is null, and the rows stay whole).
static int run_decode_plan(hkv_decode_plan *plan, const void *q, float scale, void *out, float *lse_out,
                           void *workspace, void *stream) {
    if (plan->pool->d.dtype == HKV_FP32) {
        RowsLaunch a{view_of(plan->pool), static_cast<const float *>(q), plan->d_bt, plan->d_rows_req, plan->d_rows_len,
                     static_cast<float *>(out), lse_out, plan->n_req, plan->num_q_heads, plan->max_pages, scale,
                     workspace ? plan->row_parts : 1, static_cast<float *>(workspace)};
        HKV_HIP(launch_rows_fp32(a, static_cast<hipStream_t>(stream)));
        return HKV_OK;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    // per partial: o as fp16 times a power of two, lse, and the reciprocal of that power
    uint16_t *o_parts = static_cast<uint16_t *>(workspace);
    float *lse_parts = reinterpret_cast<float *>(static_cast<char *>(workspace) +
                                                 align_up((size_t)plan->n_parts * HKV_HEAD_DIM * sizeof(uint16_t), 256));
    float *down_parts = lse_parts + align_up((size_t)plan->n_parts * sizeof(float), 256) / sizeof(float);
    const bool prof = plan->profiling;
    const bool tiles = !plan->tile_items.empty();
    const bool fork = forks(*plan);
    // The tile kernel goes first and stays on the caller's stream, so that its persistent workgroups, which need
    // a whole compute unit each, take theirs before the other kernel's many small workgroups fill the chip; that
    // kernel follows on the plan's own stream (behind an event that marks the same point of the caller's stream)
    // and is joined again before the merge.
    if (fork) {
        HKV_HIP(hipEventRecord(plan->ev_fork, s));
        HKV_HIP(hipStreamWaitEvent(plan->side, plan->ev_fork, 0));
    }
    const DecodeTilesLaunch t{view_of(plan->pool), q, plan->d_tile_items, plan->d_pages, plan->d_node_req_idx, o_parts, lse_parts,
                              down_parts, (int32_t)plan->tile_items.size(), plan->num_q_heads, plan->max_parts, scale,
                              plan->tile_workgroups, plan->d_q_rows};
    const DecodeLaunch a{view_of(plan->pool), q, plan->d_items, plan->d_pages, plan->d_node_req_idx, o_parts, lse_parts,
                         down_parts, (int32_t)plan->items.size(), plan->num_q_heads, plan->max_parts, scale,
                         plan->d_row_leaf, plan->d_row_limit, plan->d_row_mask, plan->n_single, plan->n_stages,
                         plan->fp8_matrix ? 1 : 0, plan->d_q_rows, plan->has_shared ? 1 : 0, plan->restart_tokens};
    if (plan->path_waves) {
        DecodePathLaunch p{};
        static_cast<DecodeLaunch &>(p) = a;
        p.paths = plan->d_paths;
        p.path_stride = plan->path_stride;
        p.n_paths = plan->n_paths;
        p.out = out;
        p.lse_out = lse_out;
        HKV_HIP(launch_decode_paths(p, plan->path_waves, s, prof ? plan->ev[0] : nullptr, prof ? plan->ev[1] : nullptr));
        if (prof) {
            HKV_HIP(hipEventRecord(plan->ev[2], s));
            HKV_HIP(hipEventRecord(plan->ev[3], s));
            plan->profiled_run = true;
        }
        return HKV_OK;
    }
    if (plan->fused) {
        HKV_HIP(launch_decode_fused(a, t, s, prof ? plan->ev[0] : nullptr, prof ? plan->ev[1] : nullptr));
    } else if (tiles) {
        HKV_HIP(launch_decode_tiles(t, s, prof ? plan->ev_tile[0] : nullptr, prof ? plan->ev_tile[1] : nullptr));
    }
    if (!plan->items.empty() && !plan->fused) {
        hipStream_t rs = fork ? plan->side : s;
        HKV_HIP(launch_decode(a, rs, prof ? plan->ev[0] : nullptr, prof ? plan->ev[1] : nullptr));
        if (fork) {
            HKV_HIP(hipEventRecord(plan->ev_join, plan->side));
            HKV_HIP(hipStreamWaitEvent(s, plan->ev_join, 0));
        }
    }
    HKV_HIP(launch_lse_merge_dense(o_parts, lse_parts, plan->d_part_count, plan->num_q_heads, plan->max_parts,
                                   plan->n_req * plan->num_q_heads, out, HKV_BF16, lse_out, s,
                                   prof ? plan->ev[2] : nullptr, prof ? plan->ev[3] : nullptr, plan->d_q_rows, down_parts));
    if (prof) plan->profiled_run = !plan->items.empty() || tiles;
    return HKV_OK;
}

static int check_decode_run(const hkv_decode_plan *plan, const void *q, const void *out, const char *who) {
    if (!q || !out) return fail(HKV_EINVAL, "%s: null q or out", who);
    if ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(out)) & 15)
        return fail(HKV_EINVAL, "%s: q and out must be 16-byte aligned", who);
    if (plan->pool->d.dtype == HKV_FP32 ? !plan->d_bt : !plan->dev)
        return fail(HKV_EINVAL, "%s: plan was built host-only", who);
    return HKV_OK;
}

extern "C" int attn_decode_plan_run(hkv_decode_plan *plan, const void *q, float scale, void *out, float *lse_out,
                                    void *workspace, size_t workspace_bytes, void *stream) {
    if (!plan) return fail(HKV_EINVAL, "attn_decode_plan_run: null plan");
    if (plan->n_req == 0) return HKV_OK;
    if (int rc = check_decode_run(plan, q, out, "attn_decode_plan_run")) return rc;
    const size_t need = hkv_decode_plan_workspace_bytes(plan);
    if (plan->pool->d.dtype == HKV_FP32) {  // a workspace is welcome, not needed
        const bool room = workspace && !(reinterpret_cast<uintptr_t>(workspace) & 15) && workspace_bytes >= need;
        return run_decode_plan(plan, q, scale, out, lse_out, room ? workspace : nullptr, stream);
    }
    if (need && (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255)))
        return fail(HKV_EINVAL, "attn_decode_plan_run: workspace must be non-null and 256-byte aligned");
    if (workspace_bytes < need)
        return fail(HKV_ENOMEM, "attn_decode_plan_run: workspace has %zu bytes, %zu needed", workspace_bytes, need);
    return run_decode_plan(plan, q, scale, out, lse_out, workspace, stream);
}

extern "C" size_t hkv_static_workspace_bytes(void) { return kStaticWorkspaceBytes; }

extern "C" int attn_decode_plan_run_static(hkv_decode_plan *plan, const void *q, float scale, void *out,
                                           float *lse_out, void *stream) {
    if (!plan) return fail(HKV_EINVAL, "attn_decode_plan_run_static: null plan");
    if (plan->n_req == 0) return HKV_OK;
    if (int rc = check_decode_run(plan, q, out, "attn_decode_plan_run_static")) return rc;
    if (plan->pool->d.dtype == HKV_FP32) return run_decode_plan(plan, q, scale, out, lse_out, nullptr, stream);  // (no partials: whole rows)
    const size_t need = hkv_decode_plan_workspace_bytes(plan);
    if (need > kStaticWorkspaceBytes)
        return fail(HKV_ENOMEM, "attn_decode_plan_run_static: the plan needs %zu bytes of workspace, the static "
                    "workspace holds %zu (use attn_decode_plan_run with a workspace of the caller's)", need,
                    (size_t)kStaticWorkspaceBytes);
    void *ws = nullptr;  // this device's copy of the static array (looked up when the plan was created)
    HKV_HIP(prepare_decode_device(&ws));
    return run_decode_plan(plan, q, scale, out, lse_out, ws, stream);
}

extern "C" int hkv_decode_plan_set_profiling(hkv_decode_plan *plan, int32_t mode) {
    if (!plan) return fail(HKV_EINVAL, "hkv_decode_plan_set_profiling: null plan");
    if (mode < 0 || mode > 1) return fail(HKV_EINVAL, "hkv_decode_plan_set_profiling: mode %d", mode);
    if (mode == 1 && !plan->ev[0]) {
        for (hipEvent_t &e : plan->ev) HKV_HIP(hipEventCreate(&e));
        for (hipEvent_t &e : plan->ev_tile) HKV_HIP(hipEventCreate(&e));
    }
    plan->profiling = mode == 1;
    return HKV_OK;
}

// GPU time of the node phase of the most recent profiled run: from the earlier begin to the later end of the
// kernel over `items` and the tile kernel (either may be absent), and each of the two on its own.
static int node_phase_ms(hkv_decode_plan *plan, float *span, float *rows_ms, float *tile_ms) {
    const bool rows = !plan->items.empty(), tiles = !plan->tile_items.empty() && !plan->fused;  // (one launch: its events are ev[0..1])
    *span = *rows_ms = *tile_ms = 0.f;
    if (rows) HKV_HIP(hipEventElapsedTime(rows_ms, plan->ev[0], plan->ev[1]));
    if (tiles) HKV_HIP(hipEventElapsedTime(tile_ms, plan->ev_tile[0], plan->ev_tile[1]));
    if (rows && tiles) {  // on the time line of the tile kernel's begin
        float rows_begin = 0.f, rows_end = 0.f;
        HKV_HIP(hipEventElapsedTime(&rows_begin, plan->ev_tile[0], plan->ev[0]));
        HKV_HIP(hipEventElapsedTime(&rows_end, plan->ev_tile[0], plan->ev[1]));
        *span = std::max(*tile_ms, rows_end) - std::min(0.f, rows_begin);
    } else {
        *span = rows ? *rows_ms : *tile_ms;
    }
    return HKV_OK;
}

extern "C" int hkv_decode_plan_elapsed_ms(hkv_decode_plan *plan, float *node_ms, float *merge_ms) {
    if (!plan || !node_ms || !merge_ms) return fail(HKV_EINVAL, "hkv_decode_plan_elapsed_ms: null argument");
    if (!plan->profiled_run) return fail(HKV_EINVAL, "hkv_decode_plan_elapsed_ms: no profiled run has been queued");
    HKV_HIP(hipEventSynchronize(plan->ev[3]));
    float rows_ms = 0.f, tile_ms = 0.f;
    if (int rc = node_phase_ms(plan, node_ms, &rows_ms, &tile_ms)) return rc;
    HKV_HIP(hipEventElapsedTime(merge_ms, plan->ev[2], plan->ev[3]));
    return HKV_OK;
}

extern "C" int hkv_decode_plan_elapsed_kernels_ms(hkv_decode_plan *plan, float *rows_kernel_ms, float *tile_kernel_ms) {
    if (!plan || !rows_kernel_ms || !tile_kernel_ms) return fail(HKV_EINVAL, "hkv_decode_plan_elapsed_kernels_ms: null argument");
    if (!plan->profiled_run) return fail(HKV_EINVAL, "hkv_decode_plan_elapsed_kernels_ms: no profiled run has been queued");
    HKV_HIP(hipEventSynchronize(plan->ev[3]));
    float span = 0.f;
    return node_phase_ms(plan, &span, rows_kernel_ms, tile_kernel_ms);
}

static bool same_forest(const hkv_decode_plan *pl, const hkv_node *nodes, int32_t n_nodes, const int32_t *node_pages,
                        int32_t n_node_pages, const int32_t *req_leaf, int32_t n_req, int32_t num_q_heads) {
    return pl && pl->num_q_heads == num_q_heads && (int32_t)pl->key_nodes.size() == n_nodes &&
           (int32_t)pl->key_pages.size() == n_node_pages && (int32_t)pl->req_leaf.size() == n_req &&
           (n_nodes == 0 || !memcmp(pl->key_nodes.data(), nodes, sizeof(hkv_node) * n_nodes)) &&
           (n_node_pages == 0 || !memcmp(pl->key_pages.data(), node_pages, sizeof(int32_t) * n_node_pages)) &&
           (n_req == 0 || !memcmp(pl->req_leaf.data(), req_leaf, sizeof(int32_t) * n_req));
}

static int cached_decode_plan(hkv_pool *pool, const hkv_node *nodes, int32_t n_nodes, const int32_t *node_pages,
                              int32_t n_node_pages, const int32_t *req_leaf, int32_t n_req, int32_t num_q_heads,
                              uint32_t flags, hkv_decode_plan **out) {
    if (!pool) return fail(HKV_EINVAL, "null pool");
    if (n_nodes < 0 || n_node_pages < 0 || n_req < 0 || (n_nodes > 0 && !nodes) || (n_node_pages > 0 && !node_pages) ||
        (n_req > 0 && !req_leaf))
        return fail(HKV_EINVAL, "bad forest arguments");
    hkv_decode_plan *c = pool->cached_decode;
    if (same_forest(c, nodes, n_nodes, node_pages, n_node_pages, req_leaf, n_req, num_q_heads) &&
        (c->dev || (flags & HKV_PLAN_HOST_ONLY))) {
        *out = c;
        return HKV_OK;
    }
    hkv_decode_plan *fresh = nullptr;
    if (int rc = hkv_decode_plan_create(pool, nodes, n_nodes, node_pages, n_node_pages, req_leaf, n_req, num_q_heads,
                                        flags, &fresh))
        return rc;
    if (c) hkv_decode_plan_destroy(c);
    pool->cached_decode = fresh;
    *out = fresh;
    return HKV_OK;
}

extern "C" int attn_decode_prefix_tree(hkv_pool *pool, const void *q, const hkv_node *nodes, int32_t n_nodes,
                                       const int32_t *node_pages, int32_t n_node_pages, const int32_t *req_leaf,
                                       int32_t n_req, int32_t num_q_heads, float scale, void *out, float *lse_out,
                                       void *workspace, size_t workspace_bytes, void *stream) {
    hkv_decode_plan *pl = nullptr;
    // validate everything that does not need the device before touching it
    if (n_req > 0 && (!q || !out)) return fail(HKV_EINVAL, "attn_decode_prefix_tree: null q or out");
    if (int rc = cached_decode_plan(pool, nodes, n_nodes, node_pages, n_node_pages, req_leaf, n_req, num_q_heads, 0,
                                    &pl))
        return rc;
    return attn_decode_plan_run(pl, q, scale, out, lse_out, workspace, workspace_bytes, stream);
}

extern "C" size_t attn_decode_workspace_bytes(hkv_pool *pool, const hkv_node *nodes, int32_t n_nodes,
                                              const int32_t *node_pages, int32_t n_node_pages, const int32_t *req_leaf,
                                              int32_t n_req, int32_t num_q_heads) {
    hkv_decode_plan *pl = nullptr;
    uint32_t flags = (pool && pool->cached_decode && pool->cached_decode->dev) ? 0u : (uint32_t)HKV_PLAN_HOST_ONLY;
    if (cached_decode_plan(pool, nodes, n_nodes, node_pages, n_node_pages, req_leaf, n_req, num_q_heads, flags, &pl))
        return 0;
    return hkv_decode_plan_workspace_bytes(pl);
}

// ---------------------------------------------------------------------------------------------
// prefill planning
// cu_q: request r's new tokens are rows cu_q[r] .. cu_q[r + 1] - 1 of q / out / lse.  q_row_begin (may be null):
// they are rows q_row_begin[r] .. q_row_begin[r] + (cu_q[r + 1] - cu_q[r]) - 1 instead.
//
// The tiles of a small batch, cut along their keys into equal shares of one persistent workgroup per compute unit.  All
// KV heads have the same tiles, so one head's are laid out over its n_cu / Hkv workers (workgroup index = worker * Hkv +
// head: a head stays on its XCD): whole tiles, longest first, while whole rounds of them remain, then what is left end to
// end, cut where a worker's share is full.  Taken where the estimate says so (in key blocks of 64 tokens, 1.4 us each on a
// full chip, a little less on one that is not): a tile or segment costs 4 blocks beside its own, the partials 135 KB each
// on their way through memory and the second kernel 3 more.  Against a workgroup per tile, 32 / 8 heads, one request:
// 64 / 256 / 1024 new tokens over 8192 cached ones 154 / 159 / 178 -> 32 / 47 / 141 us, 700 over 4096 94.2 -> 60.4,
// 128 over 1024 28.1 -> 21.9; six requests of 256 to 512 over 2048 106.0 -> 92.9.  Where the estimate gains less than 13 %
// it was a loss as often as not (three of 1024 over 8192: estimate 0.89, measured 0.98 to 1.01).
//
// block_cost: what a key block costs segments of such tiles, as a share of what it costs one of more than 128 rows; whole_block_cost:
// the same of whole tiles.  Returns the estimate for the way taken (0: not estimated, a workgroup per tile).
static double split_prefill_tiles(hkv_prefill_plan &pl, const std::vector<PrefillTile> &head_tiles, int n_cu, double block_cost, double whole_block_cost) {
    const int Hkv = pl.pool->d.num_kv_heads;
    const int n = (int)head_tiles.size(), workers = n_cu / Hkv;
    if (n == 0 || workers < 2 || n > 4 * workers) return 0;
    const double kOver = 4.0 / block_cost;  // (all below in blocks of these tiles)
    std::vector<int> blocks(n);
    for (int i = 0; i < n; ++i) {
        const PrefillTile &t = head_tiles[i];
        blocks[i] = (t.prefix_len + t.q_begin + t.n_q + 63) / 64;
    }
    // whole: dispatched in order, each to the workgroup that is free first
    std::vector<double> load(workers, 0.0);
    for (int i = 0; i < n; ++i) *std::min_element(load.begin(), load.end()) += blocks[i] * (whole_block_cost / block_cost) + kOver;
    const double whole_cost = *std::max_element(load.begin(), load.end());

    const int n_whole = n / workers * workers;
    std::vector<std::vector<int>> own(workers);
    std::fill(load.begin(), load.end(), 0.0);
    for (int i = 0; i < n_whole; ++i) {
        const int w = (int)(std::min_element(load.begin(), load.end()) - load.begin());
        own[w].push_back(i);
        load[w] += blocks[i] + kOver;
    }
    if (n_whole == n) return whole_cost * block_cost;  // whole rounds: nothing to gain
    int64_t rest = 0;
    for (int i = n_whole; i < n; ++i) rest += blocks[i];
    // the level up to which the rest fills the workers (a worker whose whole tiles reach it gets none), each paying one more segment
    double level = 0;
    for (double l : load) level += l;
    level = (level + rest + 1.5 * kOver * workers) / workers;
    if (level - *std::min_element(load.begin(), load.end()) < 3 * kOver) {  // shares too short: fewer, longer ones
        level = *std::min_element(load.begin(), load.end()) + 3 * kOver;
    }
    struct Cut { int tile, b0, b1; };
    std::vector<std::vector<Cut>> cuts(workers);
    int tile = n_whole, at = 0, w = 0, n_cuts = 0;
    double worst = *std::max_element(load.begin(), load.end());
    while (tile < n) {
        const bool last = w == workers - 1;
        int room = last ? 1 << 28 : (int)std::floor(level - load[w] - kOver);
        while (tile < n && (room >= 4 || room >= blocks[tile] - at)) {  // no segment below four blocks but a tile's end
            int take = std::min(room, blocks[tile] - at);
            if (blocks[tile] - at - take < 4) take = blocks[tile] - at;
            cuts[w].push_back({tile, at, at + take});
            ++n_cuts;
            load[w] += take + kOver;
            room -= take + (int)kOver;
            at += take;
            if (at == blocks[tile]) {
                ++tile;
                at = 0;
            }
        }
        worst = std::max(worst, load[w]);
        if (last) break;
        ++w;
    }
    const double split_cost = worst + (3.0 + n_cuts * (double)Hkv * kSplitPartFloats * 4 / 5e6 / 1.4) / block_cost;
    if (split_cost > 0.87 * whole_cost || (int64_t)n_cuts * Hkv > 1024) return whole_cost * block_cost;

    std::vector<int> pieces(n, 0);
    for (auto &c : cuts)
        for (const Cut &x : c) ++pieces[x.tile];
    std::vector<int32_t> part0((size_t)n * Hkv, -1), used((size_t)n * Hkv, 0);
    int32_t parts = 0;
    for (int i = n_whole; i < n; ++i)
        if (pieces[i] > 1)
            for (int h = 0; h < Hkv; ++h) {
                part0[(size_t)i * Hkv + h] = parts;
                PrefillTile t = head_tiles[i];
                t.kv_head = h;
                pl.split.push_back(PrefillSplitTile{t, parts, pieces[i]});
                parts += pieces[i];
            }
    pl.n_parts = parts;
    pl.seg_begin.push_back(0);
    for (int k = 0; k < workers; ++k)
        for (int h = 0; h < Hkv; ++h) {
            for (int i : own[k]) {
                PrefillTile t = head_tiles[i];
                t.kv_head = h;
                pl.segments.push_back(PrefillSegment{t, t.prefix_len + t.q_begin + t.n_q, -1});
                pl.seg_tile.push_back(i * Hkv + h);
            }
            for (const Cut &x : cuts[k]) {
                PrefillTile t = head_tiles[x.tile];
                const int end = t.prefix_len + t.q_begin + t.n_q;
                t.kv_head = h;
                t.prefix_len -= 64 * x.b0;  // (new tokens in front of the segment get negative positions: they see nothing of it)
                t.kv_len -= 64 * x.b0;
                t.bt_off += 4 * x.b0;
                const size_t th = (size_t)x.tile * Hkv + h;
                const int32_t part = part0[th] < 0 ? -1 : part0[th] + used[th]++;
                pl.segments.push_back(PrefillSegment{t, std::min(end, 64 * x.b1) - 64 * x.b0, part});
                pl.seg_tile.push_back((int32_t)th);
            }
            pl.seg_begin.push_back((int32_t)pl.segments.size());
        }
    return split_cost * block_cost;
}

static int create_prefill_plan(hkv_pool *pool, const int32_t *cu_q, const int32_t *q_row_begin, const int32_t *block_table,
                               int32_t max_pages, const int32_t *kv_len, int32_t n_req, int32_t num_q_heads,
                               uint32_t flags, hkv_prefill_plan **out) {
    if (!pool || !out) return fail(HKV_EINVAL, "hkv_prefill_plan_create: null argument");
    *out = nullptr;
    const int Hkv = pool->d.num_kv_heads;
    if (num_q_heads <= 0 || num_q_heads % Hkv) return fail(HKV_ESHAPE, "hkv_prefill_plan_create: %d query heads over %d KV heads", num_q_heads, Hkv);
    const int G = num_q_heads / Hkv;
    if (G > 16) return fail(HKV_ESHAPE, "hkv_prefill_plan_create: query/KV head ratio %d (supported: 1..16)", G);
    if (n_req < 0 || max_pages < 0 || (n_req > 0 && (!cu_q || !kv_len || (max_pages > 0 && !block_table))))
        return fail(HKV_EINVAL, "hkv_prefill_plan_create: bad argument");
    if (n_req > 0 && cu_q[0] != 0) return fail(HKV_EINVAL, "hkv_prefill_plan_create: cu_q[0] must be 0");
    for (int r = 0; r < n_req; ++r) {
        int64_t s = (int64_t)cu_q[r + 1] - cu_q[r];
        if (s < 0) return fail(HKV_EINVAL, "hkv_prefill_plan_create: cu_q decreases at request %d", r);
        if (kv_len[r] < s) return fail(HKV_EINVAL, "hkv_prefill_plan_create: request %d has kv_len %d < %lld new tokens", r, kv_len[r], (long long)s);
        int64_t need = ((int64_t)kv_len[r] + pool->d.page_size - 1) / pool->d.page_size;
        if (need > max_pages) return fail(HKV_ENOMEM, "hkv_prefill_plan_create: request %d needs %lld pages, max_pages is %d", r, (long long)need, max_pages);
        if (s == 0) continue;  // nothing of this request is read
        for (int64_t i = 0; i < need; ++i) {
            int32_t id = block_table[(size_t)r * max_pages + i];
            if (id < 0 || id >= pool->d.num_pages)
                return fail(HKV_ERANGE, "hkv_prefill_plan_create: request %d page %lld has id %d outside pool of %d", r, (long long)i, id, pool->d.num_pages);
        }
    }
    hkv_prefill_plan *pl = new (std::nothrow) hkv_prefill_plan;
    if (!pl) return fail(HKV_ENOMEM, "hkv_prefill_plan_create: out of host memory");
    pl->pool = pool;
    pl->n_req = n_req;
    pl->num_q_heads = num_q_heads;
    pl->key_max_pages = max_pages;
    pl->total_q = n_req ? cu_q[n_req] : 0;
    pl->cu_q.assign(cu_q, cu_q + (n_req ? n_req + 1 : 0));
    pl->kv_len.assign(kv_len, kv_len + n_req);
    if (n_req && max_pages) pl->block_table.assign(block_table, block_table + (size_t)n_req * max_pages);
    // the kernels index 16-token blocks: block j of page p is block p * S + j of the buffers
    const int S = pool->blocks_per_page;
    const int max_blocks = max_pages * S;
    pl->max_pages = max_blocks;
    std::vector<int32_t> blocks((size_t)n_req * max_blocks, 0);
    for (int r = 0; r < n_req; ++r) {
        if (cu_q[r + 1] == cu_q[r]) continue;
        const int64_t nb = ((int64_t)kv_len[r] + HKV_PAGE_SIZE - 1) / HKV_PAGE_SIZE;
        for (int64_t b = 0; b < nb; ++b)
            blocks[(size_t)r * max_blocks + b] = block_table[(size_t)r * max_pages + b / S] * S + (int32_t)(b % S);
    }
    // Tiles of one KV head, longest key range first (among equals the request's order): request r's new tokens as wholes(r) tiles of TQ
    // tokens, then the rest as tiles of `half`.
    auto head_tiles_by = [&](const int TQ, const int half, auto &&wholes) {
        struct Proto { int32_t req, q_begin, n_q; int64_t extent; };
        std::vector<Proto> protos;
        for (int r = 0; r < n_req; ++r) {
            int s = cu_q[r + 1] - cu_q[r];
            int prefix = kv_len[r] - s;
            const int n_whole = wholes(r);
            for (int q0 = 0, i = 0; q0 < s; ++i) {
                int nq = std::min(i < n_whole ? TQ : half, s - q0);
                protos.push_back({r, q0, nq, (int64_t)prefix + q0 + nq});
                q0 += nq;
            }
        }
        std::stable_sort(protos.begin(), protos.end(), [](const Proto &a, const Proto &b) { return a.extent > b.extent; });
        std::vector<PrefillTile> tiles;
        tiles.reserve(protos.size());
        for (const Proto &p : protos) {
            const int s = cu_q[p.req + 1] - cu_q[p.req];
            tiles.push_back(PrefillTile{p.req, p.q_begin, p.n_q, 0, (q_row_begin ? q_row_begin[p.req] : cu_q[p.req]) + p.q_begin, kv_len[p.req] - s,
                                        kv_len[p.req], p.req * max_blocks});
        }
        return tiles;
    };
    auto head_tiles_of = [&](const int TQ) { return head_tiles_by(TQ, TQ, [](int) { return 0; }); };
    // the KV heads of one query tile sit next to each other so that workgroup index mod num_kv_heads is the KV head (one head
    // per XCD when there are 8)
    auto of_all_heads = [&](const std::vector<PrefillTile> &head_tiles, std::vector<PrefillTile> &out) {
        for (const PrefillTile &t : head_tiles)
            for (int h = 0; h < Hkv; ++h) {
                out.push_back(t);
                out.back().kv_head = h;
            }
    };
    const std::vector<PrefillTile> head_tiles = head_tiles_of(prefill_tile_tokens(G));
    of_all_heads(head_tiles, pl->tiles);
    if (pool->d.dtype != HKV_FP32) {
        // Tiles in pieces of fewer rows where the tiles leave compute units without one, as long as every piece gets a compute unit.  A
        // wavefront without rows costs a piece nothing, and up to 64 rows run as token halves (tile_body.h) over more than
        // kPrefillHalvesTokens keys: a key block takes 1.3, 0.93 and 0.7 us for 256, 128 and 64 rows, 1, 0.72 and 0.54 of a whole tile's.  Over
        // fewer keys, as whole tiles, 64 rows take 0.64 by their blocks; the estimate counts the same start and end for all tiles, but
        // those of fewer rows are shorter, and 0.59 stands for both (17 of 70 random batches over up to 256 keys run in smaller pieces than
        // at 0.64 and take 0.96 of the time, none more than 1.009).
        // Taken where the estimate is 5 % shorter than the whole tiles', or than the split tiles' (64 rows: 6 %).  Of 220 random batches on
        // both sides of the latter lines, pieces of 128 rows take 0.65 to 0.90 of the split tiles' time up to the line, and the first
        // take longer at 3 % (1.025); pieces of 64 rows take 0.84 in the mean up to the line, the worst 1.019, and 0.92 from 6 to
        // 0 %, the worst 1.055.
        // 32 / 8 heads, whole, split, pieces of 128 and of 64 rows, us: 4 x 96 to 128 new tokens over 512 19.3, -, 15.6, 12.9; 2 x 192 to 256
        // over 1024 30.5, 27.4, 23.5, 18.3; 3 x 102 over 1600 37.9, 27.7, 29.7, 22.1; 6 x 92 over 1792 41.4, 35.3, 32.3, 45.2 (288 pieces);
        // 2 x 154 over 16 11.6, -, 9.5, 9.0; but 8 x 192 to 256 over 1024, 256 tiles, 38.0, -, 46.3, 65.4.
        const int n_cu = chip_shape().n_cu;
        const auto keys_of = [](const PrefillTile &t) { return t.prefix_len + t.q_begin + t.n_q; };
        const auto block_cost = [](int rows, int keys) { return rows > 128 ? 1.0 : rows > 64 ? 0.72 : keys > kPrefillHalvesTokens ? 0.54 : 0.59; };
        int most_rows = 0;
        for (const PrefillTile &t : head_tiles) most_rows = std::max(most_rows, t.n_q * G);
        const int most_keys = head_tiles.empty() ? 0 : keys_of(head_tiles.front());
        double best = split_prefill_tiles(*pl, head_tiles, n_cu, most_rows > 128 ? 1.0 : most_rows > 64 ? 0.72 : 0.64, block_cost(most_rows, most_keys));
        std::vector<PrefillTile> taken;
        for (const int rows : {128, 64}) {
            if (rows >= most_rows || best == 0 || rows < G) continue;
            std::vector<PrefillTile> pieces = head_tiles_of(rows / G);
            if ((int64_t)pieces.size() * Hkv > n_cu) break;
            const double cost = 4.0 + block_cost(rows, most_keys) * ((most_keys + 63) / 64);
            if (cost > (rows == 64 && taken.empty() && !pl->segments.empty() ? 0.94 : 0.95) * best) continue;
            best = cost;
            taken.swap(pieces);
        }
        // More tiles than compute units, but not a whole number of rounds: whole rounds of tiles, what is left as half tiles, where the
        // estimate is 5 % shorter.  A key block costs a half tile 0.6 of a whole one's time on a full chip (1.6 us, the power limit holds
        // the clock at 1.75 GHz), but the few whole tiles of a last round run at 2.4 GHz, 1.15 us a block, so that only the larger
        // gains are there: of 1046 random batches of one to eight rounds 79 run this way and take 0.956 of the time, none of them more than
        // 1.003 (at 3 % 130, 0.959 and six that lose over 2 %).  32 / 8 heads: 24 x 128 new tokens over 256 31.5 -> 29.9 us; 9 x 256 over 1024
        // 62.3 -> 58.5; one tile more than a whole round gains least, 11 x 200 over 1024 60.1 -> 60.0.
        const int workers = n_cu / Hkv, most = prefill_tile_tokens(G), half = 128 / G;
        if (taken.empty() && workers > 0 && half > 0 && most_rows > 128 && (int)head_tiles.size() > workers) {
            // by workgroups in order, each on the compute unit that is free first, in key blocks of whole tiles
            auto cost_of = [&](const PrefillTile &t, bool full_round) {
                return 4.0 + (t.n_q * G > 128 ? (full_round ? 1.0 : 0.85) : t.n_q * G > 64 ? 0.62 : 0.42) * ((keys_of(t) + 63) / 64);
            };
            auto rounds_of = [&](const std::vector<PrefillTile> &tiles) {
                std::vector<double> load(workers, 0.0);  // a heap, least first
                const size_t last = tiles.size() - tiles.size() % workers;
                for (size_t i = 0; i < tiles.size(); ++i) {
                    std::pop_heap(load.begin(), load.end(), std::greater<>());
                    load.back() += cost_of(tiles[i], i < last);
                    std::push_heap(load.begin(), load.end(), std::greater<>());
                }
                return *std::max_element(load.begin(), load.end());
            };
            // Half tiles come to no less than the whole ones they replace, so the best there can be is the whole tiles' cost in equal
            // shares, and in order these take no longer than that and the longest of them: batches of many rounds are not looked at further.
            double even = 0, longest = 0;
            for (size_t i = 0; i < head_tiles.size(); ++i) {
                const double cost = cost_of(head_tiles[i], i < head_tiles.size() - head_tiles.size() % workers);
                even += cost / workers;
                longest = std::max(longest, cost);
            }
            const double whole = even < 0.95 * (even + longest) ? rounds_of(head_tiles) : even;
            double least = 0.95 * (best > 0 ? std::min(best, whole) : whole);
            // a request's whole tiles, and what half tiles for the rest then come to
            std::vector<int32_t> wholes(n_req);
            auto halves_beside = [&](int r, int n) { return (std::max(0, cu_q[r + 1] - cu_q[r] - n * most) + half - 1) / half; };
            int64_t n_whole = 0;
            for (int r = 0; r < n_req; ++r) {
                const int s = cu_q[r + 1] - cu_q[r];
                wholes[r] = s / most + (s % most > half);
                n_whole += wholes[r];
            }
            // Whole tiles become two half tiles (three where a request's tokens need that: as few of these as possible), those of
            // the shortest key ranges first, until whole rounds of whole tiles are left: as many as there are, or one fewer.
            const int64_t most_rounds = n_whole / workers, least_rounds = even < least ? std::max<int64_t>(0, most_rounds - 1) : most_rounds + 1;
            for (int64_t rounds = most_rounds; rounds >= least_rounds; --rounds) {
                using Entry = std::pair<std::pair<int32_t, int32_t>, int32_t>;  // {half tiles more, keys}, request
                std::vector<Entry> heap;
                auto entry = [&](int r) { return Entry{{halves_beside(r, wholes[r] - 1) - halves_beside(r, wholes[r]), kv_len[r]}, r}; };
                for (int r = 0; r < n_req; ++r)
                    if (wholes[r] > 0) heap.push_back(entry(r));
                std::make_heap(heap.begin(), heap.end(), std::greater<>());
                for (; n_whole > rounds * workers; --n_whole) {
                    std::pop_heap(heap.begin(), heap.end(), std::greater<>());
                    const int r = heap.back().second;
                    heap.pop_back();
                    if (--wholes[r] > 0) {
                        heap.push_back(entry(r));
                        std::push_heap(heap.begin(), heap.end(), std::greater<>());
                    }
                }
                std::vector<PrefillTile> mixed = head_tiles_by(most, half, [&](int r) { return wholes[r]; });
                std::stable_partition(mixed.begin(), mixed.end(), [&](const PrefillTile &t) { return t.n_q * G > 128; });
                const double cost = rounds_of(mixed);
                if (cost >= least) continue;
                least = cost;
                taken.swap(mixed);
            }
        }
        if (!taken.empty()) {
            pl->segments.clear();
            pl->seg_begin.clear();
            pl->seg_tile.clear();
            pl->split.clear();
            pl->n_parts = 0;
            of_all_heads(taken, pl->pieces);
        }
    }
    // fp8 pools: number the pages this batch reads (first use first) and point the device table at them
    std::vector<int32_t> remapped;
    if (pool->d.dtype == HKV_FP8_E4M3) {
        std::unordered_map<int32_t, int32_t> index;
        remapped.assign(blocks.size(), 0);
        for (int r = 0; r < n_req; ++r) {
            if (cu_q[r + 1] == cu_q[r]) continue;
            const int64_t need = ((int64_t)kv_len[r] + HKV_PAGE_SIZE - 1) / HKV_PAGE_SIZE;
            for (int64_t i = 0; i < need; ++i) {
                const int32_t id = blocks[(size_t)r * max_blocks + i];
                auto it = index.find(id);
                if (it == index.end()) {
                    it = index.emplace(id, (int32_t)pl->src_pages.size()).first;
                    pl->src_pages.push_back(id);
                }
                remapped[(size_t)r * max_blocks + i] = it->second;
            }
        }
    }
    const std::vector<int32_t> &dev_table = pool->d.dtype == HKV_FP8_E4M3 ? remapped : blocks;
    const std::vector<PrefillTile> &run_tiles = pl->pieces.empty() ? pl->tiles : pl->pieces;
    if (!(flags & HKV_PLAN_HOST_ONLY) && !run_tiles.empty()) {
        size_t off_bt = align_up(sizeof(PrefillTile) * run_tiles.size(), 256);
        size_t off_src = off_bt + align_up(sizeof(int32_t) * dev_table.size(), 256);
        size_t off_fb = off_src + align_up(sizeof(int32_t) * pl->src_pages.size(), 256);
        const size_t off_seg = off_fb + 256, off_sb = off_seg + align_up(sizeof(PrefillSegment) * pl->segments.size(), 256);
        const size_t off_split = off_sb + align_up(sizeof(int32_t) * pl->seg_begin.size(), 256);
        const size_t total = off_split + align_up(sizeof(PrefillSplitTile) * pl->split.size(), 256);
        hipError_t e = hipMalloc(&pl->dev, total);
        if (e == hipSuccess) {
            char *base = static_cast<char *>(pl->dev);
            pl->d_tiles = static_cast<PrefillTile *>(pl->dev);
            pl->d_block_table = reinterpret_cast<int32_t *>(base + off_bt);
            pl->d_src_pages = reinterpret_cast<int32_t *>(base + off_src);
            pl->d_fallback = reinterpret_cast<unsigned int *>(base + off_fb);
            // one image, one copy: with a blocking copy or fill for each part a plan over split tiles took 75-89 us to create,
            // 30-38 this way, and a plan made for a single run has to gain that back
            std::vector<char> image(total, 0);
            auto put = [&](size_t off, const auto &v) { if (!v.empty()) memcpy(image.data() + off, v.data(), sizeof(v[0]) * v.size()); };
            put(0, run_tiles);
            put(off_bt, dev_table);
            put(off_src, pl->src_pages);
            if (!pl->segments.empty()) {
                pl->d_segments = reinterpret_cast<PrefillSegment *>(base + off_seg);
                pl->d_seg_begin = reinterpret_cast<int32_t *>(base + off_sb);
                pl->d_split = reinterpret_cast<PrefillSplitTile *>(base + off_split);
                put(off_seg, pl->segments);
                put(off_sb, pl->seg_begin);
                put(off_split, pl->split);
            }
            e = hipMemcpy(pl->dev, image.data(), image.size(), hipMemcpyHostToDevice);
        }
        if (e == hipSuccess && pool->d.dtype == HKV_FP32 && pl->total_q > 0) {
            std::vector<int32_t> rr(2 * (size_t)pl->total_q);
            for (int r = 0; r < n_req; ++r)
                for (int i = cu_q[r]; i < cu_q[r + 1]; ++i) {
                    rr[i] = r;
                    rr[(size_t)pl->total_q + i] = kv_len[r] - (cu_q[r + 1] - cu_q[r]) + (i - cu_q[r]) + 1;
                }
            e = hipMalloc((void **)&pl->d_rows_req, sizeof(int32_t) * rr.size());
            if (e == hipSuccess) {
                pl->d_rows_len = pl->d_rows_req + pl->total_q;
                e = hipMemcpy(pl->d_rows_req, rr.data(), sizeof(int32_t) * rr.size(), hipMemcpyHostToDevice);
            }
        }
        if (e != hipSuccess) {
            if (pl->dev) (void)hipFree(pl->dev);
            if (pl->d_rows_req) (void)hipFree(pl->d_rows_req);
            delete pl;
            return fail_hip(e, "hkv_prefill_plan_create: device upload");
        }
    }
    *out = pl;
    return HKV_OK;
}

extern "C" int hkv_prefill_plan_create(hkv_pool *pool, const int32_t *cu_q, const int32_t *block_table,
                                       int32_t max_pages, const int32_t *kv_len, int32_t n_req, int32_t num_q_heads,
                                       uint32_t flags, hkv_prefill_plan **out) {
    return create_prefill_plan(pool, cu_q, nullptr, block_table, max_pages, kv_len, n_req, num_q_heads, flags, out);
}

extern "C" int hkv_prefill_plan_create_rows(hkv_pool *pool, const int32_t *q_row_begin, const int32_t *q_len,
                                            const int32_t *block_table, int32_t max_pages, const int32_t *kv_len,
                                            int32_t n_req, int32_t num_q_heads, uint32_t flags, hkv_prefill_plan **out) {
    if (!pool || !out) return fail(HKV_EINVAL, "hkv_prefill_plan_create_rows: null argument");
    *out = nullptr;
    if (pool->d.dtype == HKV_FP32) return fail(HKV_ESHAPE, "hkv_prefill_plan_create_rows: bf16 and fp8 pools only");
    if (n_req < 0 || (n_req > 0 && (!q_row_begin || !q_len))) return fail(HKV_EINVAL, "hkv_prefill_plan_create_rows: bad argument");
    std::vector<int32_t> cu((size_t)n_req + 1, 0);
    std::vector<std::pair<int64_t, int64_t>> spans;
    for (int r = 0; r < n_req; ++r) {
        if (q_len[r] < 0 || q_row_begin[r] < 0 || (int64_t)q_row_begin[r] + q_len[r] > INT32_MAX || (int64_t)cu[r] + q_len[r] > INT32_MAX)
            return fail(HKV_EINVAL, "hkv_prefill_plan_create_rows: request %d: rows %d .. + %d", r, q_row_begin[r], q_len[r]);
        cu[r + 1] = cu[r] + q_len[r];
        if (q_len[r] > 0) spans.push_back({q_row_begin[r], (int64_t)q_row_begin[r] + q_len[r]});
    }
    std::sort(spans.begin(), spans.end());
    for (size_t i = 1; i < spans.size(); ++i)
        if (spans[i].first < spans[i - 1].second)
            return fail(HKV_EINVAL, "hkv_prefill_plan_create_rows: two requests share row %lld", (long long)spans[i].first);
    return create_prefill_plan(pool, cu.data(), q_row_begin, block_table, max_pages, kv_len, n_req, num_q_heads, flags, out);
}

extern "C" int hkv_prefill_plan_destroy(hkv_prefill_plan *plan) {
    if (!plan) return HKV_OK;
    if (plan->dev) (void)hipFree(plan->dev);
    if (plan->d_rows_req) (void)hipFree(plan->d_rows_req);
    delete plan;
    return HKV_OK;
}

extern "C" int32_t hkv_prefill_plan_num_tiles(const hkv_prefill_plan *plan) {
    return plan ? (int32_t)plan->tiles.size() : fail(HKV_EINVAL, "null plan");
}

extern "C" int32_t hkv_prefill_plan_num_pieces(const hkv_prefill_plan *plan) {
    return plan ? (int32_t)plan->pieces.size() : fail(HKV_EINVAL, "null plan");
}
extern "C" int hkv_prefill_plan_tiles(const hkv_prefill_plan *plan, int32_t *tiles_out) {
    if (!plan || !tiles_out) return fail(HKV_EINVAL, "hkv_prefill_plan_tiles: null argument");
    static_assert(sizeof(PrefillTile) == 32, "tile layout is part of the introspection contract");
    if (!plan->tiles.empty()) memcpy(tiles_out, plan->tiles.data(), sizeof(PrefillTile) * plan->tiles.size());
    return HKV_OK;
}

extern "C" int hkv_prefill_plan_fallback_tiles(hkv_prefill_plan *plan, int64_t *count) {
    if (!plan || !count) return fail(HKV_EINVAL, "hkv_prefill_plan_fallback_tiles: null argument");
    *count = 0;
    if (!plan->d_fallback) return HKV_OK;  // host-only plan, or a plan without tiles
    unsigned int n = 0;
    HKV_HIP(hipMemcpy(&n, plan->d_fallback, sizeof(n), hipMemcpyDeviceToHost));
    *count = n;
    return HKV_OK;
}

extern "C" int32_t hkv_prefill_plan_num_segments(const hkv_prefill_plan *plan) {
    return plan ? (int32_t)plan->segments.size() : fail(HKV_EINVAL, "null plan");
}

extern "C" int hkv_prefill_plan_segments(const hkv_prefill_plan *plan, int32_t *segments_out) {
    if (!plan || !segments_out) return fail(HKV_EINVAL, "hkv_prefill_plan_segments: null argument");
    static_assert(sizeof(PrefillSegment) == 40, "segment layout is part of the introspection contract");
    for (size_t w = 0; w + 1 < plan->seg_begin.size(); ++w)
        for (int32_t i = plan->seg_begin[w]; i < plan->seg_begin[w + 1]; ++i) {
            int32_t *o = segments_out + (size_t)i * 12;
            memcpy(o, &plan->segments[i], sizeof(PrefillSegment));
            o[10] = (int32_t)w;
            o[11] = plan->seg_tile[i];
        }
    return HKV_OK;
}

// The workspace: fp8 pools first the batch's pages as bf16 (K, then V), then the partials of split tiles and their flags.
static size_t prefill_pages_bytes(const hkv_prefill_plan *plan) {
    return 2 * plan->src_pages.size() * (size_t)plan->pool->d.num_kv_heads * HKV_PAGE_SIZE * HKV_HEAD_DIM * sizeof(uint16_t);
}

extern "C" size_t hkv_prefill_plan_workspace_bytes(const hkv_prefill_plan *plan) {
    if (!plan) return 0;
    return prefill_pages_bytes(plan) + (size_t)plan->n_parts * (kSplitPartFloats * sizeof(float)) + align_up(sizeof(int32_t) * plan->n_parts, 256);
}

extern "C" int attn_prefill_plan_run(hkv_prefill_plan *plan, const void *q, float scale, void *out, float *lse_out,
                                     void *stream) {
    return attn_prefill_plan_run_ws(plan, q, scale, out, lse_out, nullptr, 0, stream);
}

extern "C" int attn_prefill_plan_run_ws(hkv_prefill_plan *plan, const void *q, float scale, void *out, float *lse_out,
                                        void *workspace, size_t workspace_bytes, void *stream) {
    if (!plan) return fail(HKV_EINVAL, "attn_prefill_plan_run: null plan");
    if (plan->tiles.empty()) return HKV_OK;
    if (!q || !out) return fail(HKV_EINVAL, "attn_prefill_plan_run: null q or out");
    if ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(out)) & 15)
        return fail(HKV_EINVAL, "attn_prefill_plan_run: q and out must be 16-byte aligned");
    if (!plan->dev) return fail(HKV_EINVAL, "attn_prefill_plan_run: plan was built host-only");
    if (plan->pool->d.dtype == HKV_FP32) {  // full-precision path
        RowsLaunch r{view_of(plan->pool), static_cast<const float *>(q), plan->d_block_table, plan->d_rows_req, plan->d_rows_len,
                     static_cast<float *>(out), lse_out, plan->total_q, plan->num_q_heads, plan->max_pages, scale};
        HKV_HIP(launch_rows_fp32(r, static_cast<hipStream_t>(stream)));
        return HKV_OK;
    }
    PoolView view = view_of(plan->pool);
    if (plan->pool->d.dtype == HKV_FP8_E4M3) {  // dequantise the pages of this batch, then read the scratch pool
        const size_t need = prefill_pages_bytes(plan);
        if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255))
            return fail(HKV_EINVAL, "attn_prefill_plan_run: an fp8 pool needs a 256-byte aligned workspace of %zu bytes", need);
        if (workspace_bytes < need)
            return fail(HKV_ENOMEM, "attn_prefill_plan_run: workspace has %zu bytes, %zu needed", workspace_bytes, need);
        void *k_dst = workspace, *v_dst = static_cast<char *>(workspace) + need / 2;
        PoolDequantLaunch d{view, plan->d_src_pages, (int32_t)plan->src_pages.size(), k_dst, v_dst};
        HKV_HIP(launch_pool_dequant(d, static_cast<hipStream_t>(stream)));
        view = PoolView{k_dst, v_dst, nullptr, nullptr, view.num_kv_heads, HKV_BF16};
    }
    PrefillLaunch a{view, q, plan->d_tiles, plan->d_block_table, out, lse_out,
                    (int32_t)(plan->pieces.empty() ? plan->tiles : plan->pieces).size(), plan->num_q_heads, scale, plan->d_fallback,
                    plan->d_segments, plan->d_seg_begin, plan->d_split, nullptr, nullptr, 0, 0};
    // Split tiles need room for their partials; a caller that brings none, or only an fp8 pool's pages, gets whole tiles.
    // The room is the caller's, so that runs on different streams (of the one-shot form's cached plan too) share nothing.
    if (plan->d_segments && workspace && (reinterpret_cast<uintptr_t>(workspace) & 255) == 0 &&
        workspace_bytes >= hkv_prefill_plan_workspace_bytes(plan)) {
        a.part_data = reinterpret_cast<float *>(static_cast<char *>(workspace) + prefill_pages_bytes(plan));
        a.part_bail = reinterpret_cast<int32_t *>(a.part_data + (size_t)plan->n_parts * kSplitPartFloats);
        a.n_workers = (int32_t)plan->seg_begin.size() - 1;
        a.n_split = (int32_t)plan->split.size();
    }
    HKV_HIP(launch_prefill(a, static_cast<hipStream_t>(stream)));
    return HKV_OK;
}

extern "C" int attn_prefill_with_prefix(hkv_pool *pool, const void *q, const int32_t *cu_q, const int32_t *block_table,
                                        int32_t max_pages, const int32_t *kv_len, int32_t n_req, int32_t num_q_heads,
                                        float scale, void *out, float *lse_out, void *workspace, size_t workspace_bytes,
                                        void *stream) {
    if (!pool) return fail(HKV_EINVAL, "attn_prefill_with_prefix: null pool");
    hkv_prefill_plan *c = pool->cached_prefill;
    bool same = c && c->dev && c->n_req == n_req && c->num_q_heads == num_q_heads && c->key_max_pages == max_pages &&
                n_req > 0 && cu_q && kv_len && block_table &&
                !memcmp(c->cu_q.data(), cu_q, sizeof(int32_t) * (n_req + 1)) &&
                !memcmp(c->kv_len.data(), kv_len, sizeof(int32_t) * n_req) &&
                !memcmp(c->block_table.data(), block_table, sizeof(int32_t) * (size_t)n_req * max_pages);
    if (!same) {
        hkv_prefill_plan *fresh = nullptr;
        if (int rc = hkv_prefill_plan_create(pool, cu_q, block_table, max_pages, kv_len, n_req, num_q_heads, 0, &fresh))
            return rc;
        if (c) hkv_prefill_plan_destroy(c);
        pool->cached_prefill = c = fresh;
    }
    return attn_prefill_plan_run_ws(c, q, scale, out, lse_out, workspace, workspace_bytes, stream);
}

extern "C" size_t attn_prefill_workspace_bytes(int32_t total_q, int32_t num_q_heads) {
    (void)total_q;
    (void)num_q_heads;
    return 0;
}
