// C-ABI front end: argument validation, error reporting and dispatch to the
// gfx950 kernels.  Every check runs on the host before anything is enqueued.
#include "../../include/ragc.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <vector>

#include "ragc_internal.h"

namespace {
thread_local char g_err[512] = "";
// test overrides of the launch plan (ragc_debug_set_attn_plan); -1 / 0 = the library decides
std::atomic<int> g_force_variant{-1};
std::atomic<int> g_force_splits{0};
std::atomic<int> g_force_product{0};
}

namespace ragc {
int set_error(int code, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}
}  // namespace ragc

namespace {

int (&fail)(int, const char*, ...) = ragc::set_error;

int esize_of(int32_t dtype) { return dtype == RAGC_DTYPE_BF16 ? 2 : dtype == RAGC_DTYPE_F32 ? 4 : 0; }

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_pool(const ragc_kv_pool* pool) {
    if (!pool) return fail(RAGC_ERR_NULL, "pool is NULL");
    if (!pool->k || !pool->v) return fail(RAGC_ERR_NULL, "pool->k / pool->v is NULL");
    if (pool->block_size != RAGC_BLOCK_SIZE) return fail(RAGC_ERR_SHAPE, "block_size %d (must be 16)", pool->block_size);
    if (pool->head_dim != 64 && pool->head_dim != 128) return fail(RAGC_ERR_SHAPE, "head_dim %d (must be 64 or 128)", pool->head_dim);
    if (esize_of(pool->dtype) == 0) return fail(RAGC_ERR_SHAPE, "dtype %d unknown", pool->dtype);
    if (pool->reserved != 0) return fail(RAGC_ERR_SHAPE, "pool->reserved must be 0");
    if (pool->kv_heads <= 0 || pool->kv_heads > 65535) return fail(RAGC_ERR_SHAPE, "kv_heads %d", pool->kv_heads);
    if (pool->num_blocks <= 0) return fail(RAGC_ERR_SHAPE, "num_blocks %d", pool->num_blocks);
    const int64_t min_stride = (int64_t)pool->kv_heads * RAGC_BLOCK_SIZE * pool->head_dim;
    if (pool->block_stride_elems < min_stride)
        return fail(RAGC_ERR_SHAPE, "block_stride_elems %lld < kv_heads*16*head_dim = %lld", (long long)pool->block_stride_elems, (long long)min_stride);
    if (!aligned16(pool->k) || !aligned16(pool->v) || (pool->block_stride_elems * esize_of(pool->dtype)) % 16 != 0)
        return fail(RAGC_ERR_ALIGN, "pool planes and block stride must be 16-byte aligned");
    return RAGC_OK;
}

struct BatchInfo {
    int64_t total_new = 0;
};

// Host view of the batch metadata.  The h_* arrays of the batch are used when given; an array
// that is missing is read back from its device copy (a synchronous copy, the slow path).
struct HostMeta {
    const int32_t* prefix_len = nullptr;
    const int32_t* new_len = nullptr;
    const int32_t* new_start = nullptr;
    const int32_t* block_table = nullptr;  // may stay NULL: then block ids are not range-checked
    std::vector<int32_t> own_prefix, own_new, own_start, own_table;
};

int hip_fail(hipError_t e, const char* what) { return fail(RAGC_ERR_HIP, "%s: %s", what, hipGetErrorString(e)); }

int read_back(std::vector<int32_t>* dst, const int32_t* dev, size_t n, const char* what) {
    if (!dev) return fail(RAGC_ERR_NULL, "%s: neither the host copy nor the device array is given", what);
    dst->resize(n);
    const hipError_t e = hipMemcpy(dst->data(), dev, n * sizeof(int32_t), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(e, what);
    return RAGC_OK;
}

// want_table: read the block table back as well when no host copy is given (validation mode).
int resolve_host(const ragc_batch* b, bool want_table, HostMeta* h) {
    const size_t R = (size_t)b->num_reqs;
    h->prefix_len = b->h_prefix_len;
    h->new_len = b->h_new_len;
    h->new_start = b->h_new_start;
    h->block_table = b->h_block_table;
    if (!h->prefix_len) {
        if (int rc = read_back(&h->own_prefix, b->prefix_len, R, "prefix_len")) return rc;
        h->prefix_len = h->own_prefix.data();
    }
    if (!h->new_len) {
        if (int rc = read_back(&h->own_new, b->new_len, R, "new_len")) return rc;
        h->new_len = h->own_new.data();
    }
    if (!h->new_start) {
        if (int rc = read_back(&h->own_start, b->new_start, R, "new_start")) return rc;
        h->new_start = h->own_start.data();
    }
    if (!h->block_table && want_table) {
        if (b->table_stride <= 0) return fail(RAGC_ERR_SHAPE, "table_stride %d", b->table_stride);
        if (int rc = read_back(&h->own_table, b->block_table, R * (size_t)b->table_stride, "block_table")) return rc;
        h->block_table = h->own_table.data();
    }
    return RAGC_OK;
}

// Host-side checks of the batch metadata.  need_device: the device arrays are required.
int check_batch(const ragc_kv_pool* pool, const ragc_batch* b, bool need_device, bool want_table, HostMeta* h, BatchInfo* info) {
    if (!b) return fail(RAGC_ERR_NULL, "batch is NULL");
    if (b->num_reqs < 0 || b->num_reqs > 65535) return fail(RAGC_ERR_SHAPE, "num_reqs %d", b->num_reqs);
    if (b->num_reqs == 0) return RAGC_OK;
    if (need_device && (!b->prefix_len || !b->new_len || !b->new_start || !b->block_table))
        return fail(RAGC_ERR_NULL, "a device array of the batch is NULL");
    if (b->table_stride <= 0) return fail(RAGC_ERR_SHAPE, "table_stride %d", b->table_stride);
    if (int rc = resolve_host(b, want_table, h)) return rc;
    for (int r = 0; r < b->num_reqs; ++r) {
        const int64_t p = h->prefix_len[r], n = h->new_len[r];
        if (p < 0 || n < 0) return fail(RAGC_ERR_RANGE, "request %d: prefix_len %lld, new_len %lld", r, (long long)p, (long long)n);
        if (h->new_start[r] < 0) return fail(RAGC_ERR_RANGE, "request %d: new_start %d", r, h->new_start[r]);
        const int64_t blocks = (p + n + RAGC_BLOCK_SIZE - 1) / RAGC_BLOCK_SIZE;
        if (blocks > b->table_stride)
            return fail(RAGC_ERR_RANGE, "request %d: %lld tokens need %lld table entries, table_stride is %d", r, (long long)(p + n), (long long)blocks, b->table_stride);
        if (h->block_table) {
            const int32_t* row = h->block_table + (int64_t)r * b->table_stride;
            for (int64_t i = 0; i < blocks; ++i)
                if (row[i] < 0 || row[i] >= pool->num_blocks)
                    return fail(RAGC_ERR_RANGE, "request %d: block_table[%lld] = %d outside [0, %d)", r, (long long)i, row[i], pool->num_blocks);
        }
        info->total_new += n;
    }
    if (info->total_new > (int64_t)1 << 30) return fail(RAGC_ERR_RANGE, "sum of new_len %lld too large", (long long)info->total_new);
    return RAGC_OK;
}

// new_start must be the running sum of new_len (what the append kernel's row search assumes)
int check_packed(const ragc_batch* b, const HostMeta& h) {
    for (int r = 0; r + 1 < b->num_reqs; ++r)
        if ((int64_t)h.new_start[r + 1] != (int64_t)h.new_start[r] + h.new_len[r])
            return fail(RAGC_ERR_RANGE, "request %d: new_start[%d] = %d, expected new_start[%d] + new_len[%d] = %lld (rows must be packed in request order)",
                        r + 1, r + 1, h.new_start[r + 1], r, r, (long long)h.new_start[r] + h.new_len[r]);
    return RAGC_OK;
}

// Debug validation of what the device side cannot check: the device arrays equal their host
// copies, and (writes = true) every block that receives new tokens appears once, in one
// request, and in no request's read-only prefix.
int validate_batch(const ragc_kv_pool* pool, const ragc_batch* b, const HostMeta& h, bool writes) {
    const size_t R = (size_t)b->num_reqs;
    std::vector<int32_t> dev;
    struct { const int32_t* host; const int32_t* device; size_t n; const char* name; } arrays[] = {
        {b->h_prefix_len, b->prefix_len, R, "prefix_len"},
        {b->h_new_len, b->new_len, R, "new_len"},
        {b->h_new_start, b->new_start, R, "new_start"},
    };
    for (auto& a : arrays) {
        if (!a.host || !a.device) continue;  // nothing to compare (a missing host copy was read from the device anyway)
        if (int rc = read_back(&dev, a.device, a.n, a.name)) return rc;
        for (size_t i = 0; i < a.n; ++i)
            if (dev[i] != a.host[i]) return fail(RAGC_ERR_RANGE, "%s[%zu]: device copy %d differs from host copy %d", a.name, i, dev[i], a.host[i]);
    }
    if (b->h_block_table && b->block_table) {
        if (int rc = read_back(&dev, b->block_table, R * (size_t)b->table_stride, "block_table")) return rc;
        for (size_t r = 0; r < R; ++r) {
            const int64_t blocks = ((int64_t)h.prefix_len[r] + h.new_len[r] + RAGC_BLOCK_SIZE - 1) / RAGC_BLOCK_SIZE;
            for (int64_t i = 0; i < blocks; ++i) {
                const size_t at = r * (size_t)b->table_stride + (size_t)i;
                if (dev[at] != b->h_block_table[at])
                    return fail(RAGC_ERR_RANGE, "block_table[%zu][%lld]: device copy %d differs from host copy %d", r, (long long)i, dev[at], b->h_block_table[at]);
            }
        }
    }
    if (!writes || !h.block_table) return RAGC_OK;
    // owner[block]: -1 untouched, r >= 0: receives new tokens of request r, -2: read as prefix by some request
    std::vector<int32_t> owner((size_t)pool->num_blocks, -1);
    for (size_t r = 0; r < R; ++r) {  // pass 1: write targets
        const int64_t p = h.prefix_len[r], n = h.new_len[r];
        if (n == 0) continue;
        const int32_t* row = h.block_table + r * (size_t)b->table_stride;
        for (int64_t i = p / RAGC_BLOCK_SIZE; i < (p + n + RAGC_BLOCK_SIZE - 1) / RAGC_BLOCK_SIZE; ++i) {
            if (owner[row[i]] != -1)
                return fail(RAGC_ERR_RANGE, "block %d receives new tokens of request %zu (table entry %lld) and of request %d: append targets must be exclusive",
                            row[i], r, (long long)i, owner[row[i]]);
            owner[row[i]] = (int32_t)r;
        }
    }
    for (size_t r = 0; r < R; ++r) {  // pass 2: read-only prefix blocks (whole blocks below the first write target)
        const int32_t* row = h.block_table + r * (size_t)b->table_stride;
        const int64_t full = (h.new_len[r] == 0 ? ((int64_t)h.prefix_len[r] + RAGC_BLOCK_SIZE - 1) : (int64_t)h.prefix_len[r]) / RAGC_BLOCK_SIZE;
        for (int64_t i = 0; i < full; ++i)
            if (owner[row[i]] >= 0)
                return fail(RAGC_ERR_RANGE, "block %d is read as cached prefix by request %zu (table entry %lld) and receives new tokens of request %d",
                            row[i], r, (long long)i, owner[row[i]]);
    }
    return RAGC_OK;
}

ragc::PagedBatch make_paged(const ragc_kv_pool* pool, const ragc_batch* b) {
    ragc::PagedBatch pb;
    pb.pool_k = pool->k;
    pb.pool_v = pool->v;
    pb.block_stride = pool->block_stride_elems;
    pb.prefix_len = b->prefix_len;
    pb.new_len = b->new_len;
    pb.new_start = b->new_start;
    pb.block_table = b->block_table;
    pb.table_stride = b->table_stride;
    pb.num_reqs = b->num_reqs;
    pb.kv_heads = pool->kv_heads;
    pb.head_dim = pool->head_dim;
    return pb;
}

// compute units of the current device (queried once per thread)
int cu_count() {
    thread_local int cus = 0;
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
            cus = n;
        else
            cus = 256;
    }
    return cus;
}

// How the bf16 path will run a batch: which kernel, on row tiles of how many rows, with how many copies of
// each item along its keys; and the workspace of the copies' partial results (0 without copies).
// ragc_prefill_attn_workspace and ragc_prefill_attn both call this, so they always agree.
struct Bf16Plan {
    std::vector<int32_t> order;  // requests with new tokens, most keys first
    bool rows_kernel = false;    // attn_bf16_rows_kernel
    int rows = ragc::kAttnRowsPerItem;
    int splits = 1;
    int waves = 8;                             // per workgroup of attn_bf16_rows_kernel
    int variant = ragc::kAttnVariantOneGroup;  // of attn_bf16_kernel
    bool quarters = false;                     // of attn_bf16_kernel: 16x16x32 products
    int64_t workspace = 0;
};

// rows: a power of two (a shift instead of a division: every request of a batch comes by here three times)
inline int64_t row_tiles(const HostMeta& h, int r, int group, int rows) {
    return ((int64_t)h.new_len[r] * group + rows - 1) >> __builtin_ctz((unsigned)rows);
}

// Requests with the most keys first, and the row tiles of one request next to each other: long items start
// early, and the workgroups that run at the same time on an XCD walk the key tiles of the same few requests at
// about the same pace, so a tile fetched by one row tile is still in that XCD's L2 for the others.
void order_requests(const HostMeta& h, int num_reqs, std::vector<int32_t>* order) {
    // one number per request, the one with the most keys smallest, then by request (at most 65535 of them); batches of
    // one length, or already in order, are left as they are
    constexpr int kSmall = 128;
    uint64_t small[kSmall];
    std::vector<uint64_t> large;
    uint64_t* rank = small;
    if (num_reqs > kSmall) {
        large.resize(num_reqs);
        rank = large.data();
    }
    int n = 0;
    bool sorted = true;
    for (int r = 0; r < num_reqs; ++r) {
        if (h.new_len[r] <= 0) continue;
        rank[n] = ((uint64_t)UINT32_MAX - ((uint32_t)h.prefix_len[r] + (uint32_t)h.new_len[r])) << 16 | (uint64_t)r;
        sorted = sorted && (n == 0 || rank[n - 1] < rank[n]);
        ++n;
    }
    if (!sorted) std::sort(rank, rank + n);
    order->resize(n);
    for (int i = 0; i < n; ++i) (*order)[i] = (int32_t)(rank[i] & 0xffff);
}

int plan_bf16(const ragc_kv_pool* pool, const ragc_batch* batch, const HostMeta& h, int group, uint32_t flags, Bf16Plan* plan) {
    int64_t items = 0, short_items = 0, max_rows = 0, max_keys = 0, req_keys = 0, sum_keys = 0;  // sum_keys: over the 32-row items
    for (int r = 0; r < batch->num_reqs; ++r) {
        const int64_t tiles = row_tiles(h, r, group, ragc::kAttnRowsPerItem);
        if (tiles > 65535) return fail(RAGC_ERR_RANGE, "request %d: new_len * group too large", r);
        if (tiles == 0) continue;
        items += tiles;
        const int64_t short_tiles = row_tiles(h, r, group, ragc::kAttnShortRows);
        short_items += short_tiles;
        const int64_t keys = (int64_t)h.prefix_len[r] + h.new_len[r];
        req_keys += keys;
        sum_keys += short_tiles * keys;
        max_rows = std::max(max_rows, (int64_t)h.new_len[r] * group);
        max_keys = std::max(max_keys, keys);
    }
    order_requests(h, batch->num_reqs, &plan->order);
    if (items == 0) return 0;
    const int64_t cus = cu_count();
    const int64_t wgs = items * pool->kv_heads, short_wgs = short_items * pool->kv_heads;
    const bool d128 = pool->head_dim == 128;
    const int force_splits = std::min(g_force_splits.load(std::memory_order_relaxed), ragc::kAttnMaxSplits);
    const int force_variant = g_force_variant.load(std::memory_order_relaxed);
    const bool may_split = !(flags & RAGC_ATTN_NO_SPLIT);
    const auto make = [&](bool rows_kernel, int64_t splits, int64_t all_items) {
        plan->rows_kernel = rows_kernel;
        plan->rows = rows_kernel ? ragc::kAttnShortRows : ragc::kAttnRowsPerItem;
        plan->splits = (int)splits;
        if (splits > 1) plan->workspace = all_items * splits * pool->kv_heads * ragc::attn_partial_bytes(pool->head_dim, plan->rows);
        return 0;
    };
    const auto rows32 = [&](int64_t splits, int waves) {
        plan->waves = waves;
        return make(true, splits, short_items);
    };
    const auto rows128 = [&](int64_t splits, int variant) {
        plan->variant = splits > 1 ? ragc::kAttnVariantOneGroup : variant;
        // Launches that the power limit holds back take the product of less energy per flop, others the one of fewer cycles
        // (attn_bf16.hip has both sides).
        const int force_product = g_force_product.load(std::memory_order_relaxed);
        plan->quarters = d128 && splits == 1 &&
                         (force_product ? force_product == 16 : sum_keys * pool->kv_heads >= (wgs >= 3 * cus ? 1500 : 12000) * cus);
        return make(false, splits, items);
    };
    // Copies that give every CU a 128-row item with at least three 64-key tiles.  Those of 32-row items (below) never take
    // more workspace.
    const int64_t splits128 = may_split ? std::max<int64_t>(1, std::min({cus / wgs, (int64_t)ragc::kAttnMaxSplits, (max_keys + 63) / 64 / 3})) : 1;

    if (force_variant >= 0 || (may_split && force_splits > 0)) {  // tests
        const int64_t splits = may_split && force_splits > 0 ? force_splits : 1;
        if (max_rows <= ragc::kAttnShortRows || (splits > 1 && force_variant != ragc::kAttnVariantOneGroup))
            return rows32(splits, force_variant == ragc::kAttnVariantOneGroup && splits == 1 ? 4 : 8);
        return rows128(splits, force_variant >= 0 ? force_variant : wgs >= 2 * cus ? ragc::kAttnVariantOneGroup : ragc::kAttnVariantTwoGroups);
    }

    // The lines below: 3600 batches, each timed with every choice; both sides of a line as the library would run them.
    const bool uniform = sum_keys * 100 >= max_keys * short_items * 97;   // every request about as long as the longest
    const bool even = sum_keys * 100 >= max_keys * short_items * 78;
    const bool many_keys = sum_keys >= 1024 * short_items;
    // The 32-row kernel takes launches of at most 32 rows per request, and those that leave CUs without a 128-row item, or a
    // second round of 128-row items half empty, as long as its own workgroups need at most two rounds (one per CU at a time at
    // head_dim 128): with fewer 128-row items than CUs 0.4-1.0 times the time of the other kernel (one request of 1000 + 256
    // tokens 14.7 us against 19.1), with one to two per CU 0.7 (416 workgroups of 272 keys 10.7 us against 16.6).  With exactly
    // one 128-row item per CU there is no second round (424 workgroups of 1811 keys: 53.7 us against 49.7).
    // At head_dim 64 several of its four-wave workgroups fit a CU next to each other, and it takes ragged batches as well:
    // with at most two 128-row items per CU the 128-row kernel takes as long as its longest item, the 32-row kernel as
    // long as its workgroups take in all, and the latter is less while their keys, per CU, are at most twice those of the
    // longest request (in these units 1.6: 19.5 us against 24.4, 2.0: 20.3 against 23.5, 2.5: 24.7 against 24.4, 3: 28.6
    // against 26.1).  At head_dim 128 it loses at 1.6 already (45.8 against 42.5).
    const bool rows_kernel = max_rows <= ragc::kAttnShortRows || (wgs != cus && wgs < 2 * cus && short_wgs <= 2 * cus) ||
                             (!d128 && wgs < 2 * cus && sum_keys * pool->kv_heads <= 2 * cus * max_keys);
    if (!rows_kernel) {
        // With at least two 128-row items per CU two 4-wave workgroups share a CU; otherwise one 8-wave workgroup divides its
        // key tiles between two wave groups.  Between one and two items per CU the second round of 8-wave workgroups costs as
        // much as the first; where the items are half empty (at most three 32-row workgroups per CU) and short, sharing is
        // faster at head_dim 128: 0.67 times up to 300 keys, 0.77 up to 600, 0.82 up to 1024 (medians of 266 batches; the
        // 32-row kernel 0.74 / 0.85 / 1.0 of its time the other way round).
        const bool shared = wgs >= 2 * cus || (d128 && wgs > cus && short_wgs <= 3 * cus && max_keys <= 1024);
        return rows128(1, shared ? ragc::kAttnVariantOneGroup : ragc::kAttnVariantTwoGroups);
    }
    // Decode steps of head_dim 64, all of one length, a little over two workgroups per CU: the four waves of a 128-row item
    // share its copies (528 of 4030 keys: 105 us against 113; medians 0.95 up to 2.5 per CU, 1.0 above).
    if (!d128 && max_rows <= ragc::kAttnShortRows && uniform && max_keys >= 300 && short_wgs > 2 * cus && 2 * short_wgs <= 5 * cus)
        return rows128(1, ragc::kAttnVariantOneGroup);
    // Workgroup ids go round-robin over the XCDs, kv head first, copies next, row tiles last: the row tiles of a request read
    // its keys through one L2 where heads times copies is a multiple of 8, and otherwise through up to `step` of them, `again`
    // bytes more from memory.
    const int64_t step = pool->kv_heads % 8 == 0 ? 1 : pool->kv_heads % 4 == 0 ? 2 : pool->kv_heads % 2 == 0 ? 4 : 8;
    const int64_t reqs = (int64_t)plan->order.size();
    const int64_t again = req_keys * pool->kv_heads * pool->head_dim * 4 / reqs * (std::min(short_items, step * reqs) - reqs);
    if (short_wgs <= cus) {
        // Copies until every CU has a workgroup, of at least two 32-key tiles for each of its eight waves; up to 1408
        // keys one copy of the whole range and no merge pass is faster (1280-1400 keys: 0.88 times at head_dim 128, 0.80 at
        // 64; 4096 keys, 8 copies: 17.9 us against 26.9).
        const int64_t tiles = (max_keys + 31) / 32;
        int64_t splits = 1;
        if (splits128 > 1 && tiles > 44)
            splits = std::max<int64_t>(1, std::min({items * splits128 * 4 / short_items, cus / short_wgs, tiles / 16, (int64_t)ragc::kAttnMaxSplits}));
        // Where `again` bytes cost time (head_dim 128, above 30 MB) the copies are made a multiple of `step`, or, where that
        // does not fit, long requests are split as 128-row items, which read their keys a quarter as often: 48 workgroups of
        // 6850 keys, 2 heads: 4 copies 19.9 us, 5 copies 31.0; without such a number the 128-row items take 0.7-1.0 times
        // the time from 60 MB on, or from 30 with up to 96 workgroups, and 1.0-1.2 times below; next to it only where it
        // leaves CUs idle: 68 of 8088 keys 40.6 against 48.8, 48 of 3509 17.0 against 15.5.
        if (d128 && splits128 > 1 && tiles > 44 && again > 30000000) {
            if (splits >= step) splits -= splits % step;
            if (splits >= step ? again > 60000000 && short_wgs * splits <= 160 : again > 60000000 || short_wgs <= 96)
                return rows128(splits128, ragc::kAttnVariantTwoGroups);
        }
        return rows32(splits, 8);
    }
    // Between one and two 32-row workgroups per CU at head_dim 128, all requests of one length: two rounds, the second more or
    // less empty.  Long ones are split as 128-row items, or take them whole where there is nothing to split and the second
    // round is short: 280 workgroups of 6025 keys 48.3 us against 68.8, 288 of 4491 40.7 against 54.0; but 492 of 6277, not
    // split, 92.2 against 78.0.  From 2200 keys on where the items are ragged or few (272 of 2946 60 against 70); with fewer
    // keys the four waves below are faster (288 of 1891: 26.5 against 29.1, medians 0.8-0.9), unless they read much again
    // (272 of 1710, 4 heads: 24.1 against 29.7).
    if (d128 && wgs < cus && max_rows > ragc::kAttnShortRows && uniform && (splits128 > 1 || short_wgs * 5 <= cus * 9) &&
        (max_keys > 3000 || again > 55000000 || (max_keys > 2200 && (splits128 >= 3 || short_wgs * 4 < wgs * 11))))
        return rows128(splits128, ragc::kAttnVariantTwoGroups);
    // Four waves per workgroup: a CU then holds two workgroups at a time at head_dim 128 (four at 64), one streams while the
    // other starts, and requests of like length do not wait for a second round.  Eight finish a long request sooner where
    // the lengths differ.  head_dim 128, 257-512 workgroups: four take 0.7-0.9 times the time up to 2200 keys, 0.9 above
    // with a mean of at least 0.78 of the longest, 1.05-1.14 below that (64 decode requests of 512-2048 keys, 8 heads: 64 us
    // against 61).  head_dim 64: 0.96 for decode steps of one length, 1.0 otherwise; above two per CU 0.9 whatever the keys.
    const bool four = d128 ? !many_keys || even || (max_rows > ragc::kAttnShortRows && max_keys <= 2200)
                           : !many_keys || short_wgs > 2 * cus || (uniform && max_rows <= ragc::kAttnShortRows);
    return rows32(1, four ? 4 : 8);
}

constexpr uint32_t kAttnFlags = RAGC_ATTN_APPEND_FUSED | RAGC_ATTN_NO_SPLIT | RAGC_ATTN_VALIDATE;

// Enqueues `launch(list, entries)` for the requests of `order`, as many per launch as the kernel arguments and a grid hold.
template <class Launch>
int run_list(const ragc::AttnLaunch& a, const HostMeta& h, const std::vector<int32_t>& order, int rows, int splits, const Launch& launch) {
    // the kernels divide workgroup ids by head_div with a multiply that is exact below 2^32 / head_div
    const int64_t max_workgroups = std::min<int64_t>(ragc::kAttnMaxWorkgroups, UINT32_MAX / a.head_div);
    const int64_t per_launch = std::max<int64_t>(1, max_workgroups / ((int64_t)a.kv_heads * splits)) * splits;
    int64_t slots = 0;
    for (size_t i = 0; i < order.size(); i += ragc::kAttnMaxReqs) {
        ragc::AttnWork wk;
        wk.n_reqs = (int32_t)std::min<size_t>(ragc::kAttnMaxReqs, order.size() - i);
        wk.splits = splits;
        wk.part_base = (int32_t)slots;
        int64_t items = 0;
        for (int j = 0; j < wk.n_reqs; ++j) {
            const int r = order[i + j];
            wk.first[j] = (int32_t)items;
            wk.req[j] = {h.prefix_len[r], h.new_len[r], h.new_start[r], r};
            items += row_tiles(h, r, a.group, rows);
            if (items * splits > INT32_MAX) return fail(RAGC_ERR_RANGE, "new_len * group of the batch too large");
        }
        for (int j = wk.n_reqs; j % ragc::kAttnReqStep; ++j) wk.first[j] = INT32_MAX;
        const int64_t entries = items * splits;
        for (int64_t e0 = 0; e0 < entries; e0 += per_launch) {
            wk.entry0 = (int32_t)e0;
            const hipError_t e = launch(wk, (int)std::min<int64_t>(per_launch, entries - e0));
            if (e != hipSuccess) return fail(RAGC_ERR_HIP, "prefill attention launch: %s (earlier launches of this call stay enqueued)", hipGetErrorString(e));
        }
        slots += entries;
    }
    return RAGC_OK;
}

int run_bf16_plan(const ragc::AttnLaunch& a, const HostMeta& h, const Bf16Plan& plan, hipStream_t s) {
    return run_list(a, h, plan.order, plan.rows, plan.splits, [&](const ragc::AttnWork& wk, int entries) {
        hipError_t e = plan.rows_kernel ? ragc::launch_attn_bf16_rows(a, wk, entries, plan.waves, s) : ragc::launch_attn_bf16(a, wk, entries, plan.variant, plan.quarters, s);
        if (e == hipSuccess && wk.splits > 1) e = ragc::launch_attn_bf16_merge(a, wk, entries, plan.rows, s);
        return e;
    });
}

// fp32 path: which kernel (rows per item), and how many waves per workgroup.
// Waves: with at most one workgroup per CU eight, so that every SIMD still has two to overlap (16-row items: 256 workgroups of
// ~1100 keys 31 us against 37); with more, four, and two workgroups share a CU (416 of ~1000 keys: 45 us against 49, 512 of
// ~1100: 53 against 58; 32-row items: 848 66 against 74, 384 22 against 27).
// The 32-row items, whose kernel multiplies on the bf16 cores, take 0.72-0.85 of the time of the 16-row items where those leave
// no CU idle, and more where they do (125 of ~2000 keys: 52 us against 41) or where their rows would be half empty (320
// against 480: 15.2 against 11.9).  Lines from 160 batches timed with every choice, in workgroups of 16 rows per CU:
// head_dim 128, from 1.25 on (1.3: 0.76-0.93; 1.03-1.16: 1.0-1.2).  While they are at most one per CU, with at least 96 keys on
// average (1.6: 1.06 and 1.09 below); above, where they need fewer rounds of two per CU (another 65 batches: 264 against 504
// 14.7 us against 12.2, 288 against 504 of ~1270 keys 76 against 61, 544 against 1016 1.04, but 328 against 656 0.90).
// head_dim 64, whose steps are shorter, from 1 to 2 with at least 200 keys (0.74-0.96), and from 4.5 on with at least 96 keys
// (0.74-0.94), or where they need fewer rounds, three per CU and four (712 against 1240 of 14 keys 0.91; 864 against 1440 of 10
// 1.14); 2 to 4: 0.93-1.11.
struct F32Plan {
    int rows, waves;
};
F32Plan plan_f32(const HostMeta& h, const std::vector<int32_t>& order, int group, int kv_heads, int head_dim) {
    int64_t tiles = 0, split_tiles = 0, keys = 0;  // keys: over the 16-row items
    for (int r : order) {
        const int64_t t = row_tiles(h, r, group, ragc::kAttnF32Rows);
        tiles += t;
        split_tiles += row_tiles(h, r, group, ragc::kAttnF32SplitRows);
        keys += t * ((int64_t)h.prefix_len[r] + h.new_len[r]);
    }
    const int64_t cus = cu_count(), wgs = tiles * kv_heads, split_wgs = split_tiles * kv_heads;
    const auto fewer_rounds = [&](int64_t at_once, int64_t split_at_once) {
        return (split_wgs + split_at_once - 1) / split_at_once < (wgs + at_once - 1) / at_once;
    };
    const bool split = split_tiles * 5 <= tiles * 3 &&
                       (head_dim == 128 ? wgs * 4 >= cus * 5 && (split_wgs > cus ? fewer_rounds(2 * cus, 2 * cus) : keys >= 96 * tiles)
                                        : (wgs * 2 >= cus * 9 && (keys >= 96 * tiles || fewer_rounds(4 * cus, 3 * cus))) ||
                                              (wgs > cus && split_wgs <= cus && keys >= 200 * tiles));
    return {split ? ragc::kAttnF32SplitRows : ragc::kAttnF32Rows, (split ? split_wgs : wgs) > cus ? 4 : 8};
}

int run_f32(const ragc::AttnLaunch& a, const ragc_batch* batch, const HostMeta& h, hipStream_t s) {
    std::vector<int32_t> order;
    order_requests(h, batch->num_reqs, &order);
    const F32Plan plan = plan_f32(h, order, a.group, a.kv_heads, a.head_dim);
    return run_list(a, h, order, plan.rows, 1,
                    [&](const ragc::AttnWork& wk, int entries) { return ragc::launch_attn_f32(a, wk, entries, plan.rows, plan.waves, s); });
}

// ---- partial results of key-split work items for callers that cannot allocate --------------
// One array per GPU (every device that loads the library holds its own copy until the process
// ends).  Host code must never pass the array's name to a kernel: that name is a host-side
// stand-in; the device address comes from hipGetSymbolAddress, once per device.
constexpr int64_t kStaticScratchBytes = 256 * 128 * (128 + 2) * 4;  // 256 partial results at head_dim 128: 17,039,360 bytes
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

int static_scratch(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(RAGC_ERR_RANGE, "device ordinal %d outside [0, %d)", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));  // address of THIS device's copy
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        if (!p || (reinterpret_cast<uintptr_t>(p) & 255u)) return fail(RAGC_ERR_ALIGN, "static scratch is not 256-byte aligned");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return RAGC_OK;
}

int prefill_attn_impl(const ragc_kv_pool* pool, const ragc_batch* batch, const void* q, const void* k_new,
                      const void* v_new, void* out, int32_t q_heads, float softmax_scale, uint32_t flags,
                      void* workspace, size_t workspace_bytes, bool use_static_scratch, void* stream) {
    g_err[0] = 0;
    if (int rc = check_pool(pool)) return rc;
    if (flags & ~kAttnFlags) return fail(RAGC_ERR_SHAPE, "unknown flags 0x%x", flags);
    if (q_heads <= 0 || q_heads % pool->kv_heads != 0)
        return fail(RAGC_ERR_SHAPE, "q_heads %d not a multiple of kv_heads %d", q_heads, pool->kv_heads);
    if (!(softmax_scale > 0.f) || !std::isfinite(softmax_scale))
        return fail(RAGC_ERR_SHAPE, "softmax_scale must be positive and finite");
    const bool validate = (flags & RAGC_ATTN_VALIDATE) != 0;
    if (use_static_scratch) {
        // nothing in this mode may allocate or synchronise: no read-backs
        if (validate) return fail(RAGC_ERR_SHAPE, "RAGC_ATTN_VALIDATE reads device arrays back; not available in ragc_prefill_attn_static");
        if (batch && batch->num_reqs > 0 && (!batch->h_prefix_len || !batch->h_new_len || !batch->h_new_start))
            return fail(RAGC_ERR_NULL, "ragc_prefill_attn_static needs h_prefix_len, h_new_len and h_new_start");
    }
    BatchInfo info;
    HostMeta h;
    if (int rc = check_batch(pool, batch, true, validate, &h, &info)) return rc;
    if (batch->num_reqs == 0 || info.total_new == 0) return RAGC_OK;
    if (!q || !k_new || !v_new || !out) return fail(RAGC_ERR_NULL, "q / k_new / v_new / out is NULL");
    if (!aligned16(q) || !aligned16(k_new) || !aligned16(v_new) || !aligned16(out))
        return fail(RAGC_ERR_ALIGN, "q / k_new / v_new / out must be 16-byte aligned");
    if (validate)
        if (int rc = validate_batch(pool, batch, h, (flags & RAGC_ATTN_APPEND_FUSED) != 0)) return rc;

    const auto magic = [](uint32_t d) { return d == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); };
    ragc::AttnLaunch a;
    a.pool_k = pool->k;
    a.pool_v = pool->v;
    a.block_stride = pool->block_stride_elems;
    a.block_table = batch->block_table;
    a.q = q;
    a.k_new = k_new;
    a.v_new = v_new;
    a.out = out;
    a.partial = nullptr;
    a.table_stride = batch->table_stride;
    a.kv_heads = pool->kv_heads;
    a.head_dim = pool->head_dim;
    a.q_heads = q_heads;
    a.group = q_heads / pool->kv_heads;
    a.group_magic = magic(a.group);
    a.scale_log2e = softmax_scale * 1.44269504088896340736f;
    a.fused_append = (flags & RAGC_ATTN_APPEND_FUSED) ? 1 : 0;
    a.head_shift = pool->kv_heads % 8 == 0 ? 3 : 0;
    a.head_div = (uint32_t)pool->kv_heads >> a.head_shift;
    a.head_magic = magic(a.head_div);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (pool->dtype == RAGC_DTYPE_F32) {
        return run_f32(a, batch, h, s);
    }
    Bf16Plan plan;
    if (int rc = plan_bf16(pool, batch, h, a.group, flags, &plan)) return rc;
    if (plan.workspace > 0) {
        if (use_static_scratch) {
            if (plan.workspace > kStaticScratchBytes)
                return fail(RAGC_ERR_WORKSPACE, "this batch needs %lld bytes for its partial results; the static scratch holds %lld",
                            (long long)plan.workspace, (long long)kStaticScratchBytes);
            if (int rc = static_scratch(&a.partial)) return rc;
        } else {
            if (!workspace || (int64_t)workspace_bytes < plan.workspace)
                return fail(RAGC_ERR_WORKSPACE, "workspace of %lld bytes needed (ragc_prefill_attn_workspace), %zu given",
                            (long long)plan.workspace, workspace_bytes);
            if (reinterpret_cast<uintptr_t>(workspace) & 255u) return fail(RAGC_ERR_ALIGN, "workspace must be 256-byte aligned");
            a.partial = workspace;
        }
    }
    return run_bf16_plan(a, h, plan, s);
}

}  // namespace

extern "C" {

int ragc_version(void) { return 100; }

const char* ragc_last_error(void) { return g_err; }

int64_t ragc_kv_bytes_per_token(int32_t layers, int32_t kv_heads, int32_t head_dim, int32_t dtype) {
    const int es = esize_of(dtype);
    if (layers <= 0 || kv_heads <= 0 || head_dim <= 0 || es == 0) return 0;
    return (int64_t)2 * layers * kv_heads * head_dim * es;
}

int ragc_debug_set_attn_plan(int32_t variant, int32_t splits) {
    g_err[0] = 0;
    if (variant < -1 || variant >= ragc::kAttnVariantCount) return fail(RAGC_ERR_SHAPE, "variant %d unknown", variant);
    if (splits < 0 || splits > ragc::kAttnMaxSplits) return fail(RAGC_ERR_SHAPE, "splits %d outside [0, %d]", splits, ragc::kAttnMaxSplits);
    g_force_variant.store(variant, std::memory_order_relaxed);
    g_force_splits.store(splits, std::memory_order_relaxed);
    return RAGC_OK;
}

int ragc_debug_get_attn_plan(const ragc_kv_pool* pool, const ragc_batch* batch, int32_t q_heads, uint32_t flags, int32_t* plan) {
    g_err[0] = 0;
    if (int rc = check_pool(pool)) return rc;
    if (flags & ~kAttnFlags) return fail(RAGC_ERR_SHAPE, "unknown flags 0x%x", flags);
    if (q_heads <= 0 || q_heads % pool->kv_heads != 0)
        return fail(RAGC_ERR_SHAPE, "q_heads %d not a multiple of kv_heads %d", q_heads, pool->kv_heads);
    if (!plan) return fail(RAGC_ERR_NULL, "plan is NULL");
    BatchInfo info;
    HostMeta h;
    if (int rc = check_batch(pool, batch, false, false, &h, &info)) return rc;
    plan[0] = plan[1] = plan[2] = 0;
    if (batch->num_reqs == 0 || info.total_new == 0) return RAGC_OK;
    const int group = q_heads / pool->kv_heads;
    if (pool->dtype == RAGC_DTYPE_F32) {
        std::vector<int32_t> order;
        order_requests(h, batch->num_reqs, &order);
        const F32Plan p = plan_f32(h, order, group, pool->kv_heads, pool->head_dim);
        plan[0] = p.rows;
        plan[1] = p.waves;
        plan[2] = 1;
        return RAGC_OK;
    }
    Bf16Plan p;
    if (int rc = plan_bf16(pool, batch, h, group, flags, &p)) return rc;
    plan[0] = p.rows;
    plan[1] = p.rows_kernel ? p.waves : p.variant == ragc::kAttnVariantTwoGroups ? 8 : 4;
    plan[2] = p.splits;
    return RAGC_OK;
}

int ragc_debug_set_attn_product(int32_t rows) {
    g_err[0] = 0;
    if (rows != 0 && rows != 16 && rows != 32) return fail(RAGC_ERR_SHAPE, "products of %d rows unknown", rows);
    g_force_product.store(rows, std::memory_order_relaxed);
    return RAGC_OK;
}

int ragc_debug_get_attn_product(const ragc_kv_pool* pool, const ragc_batch* batch, int32_t q_heads, uint32_t flags) {
    int32_t plan[3];
    if (int rc = ragc_debug_get_attn_plan(pool, batch, q_heads, flags, plan)) return rc;
    if (pool->dtype != RAGC_DTYPE_BF16 || pool->head_dim != 128 || plan[0] != ragc::kAttnRowsPerItem || plan[2] != 1) return 0;
    BatchInfo info;
    HostMeta h;
    if (int rc = check_batch(pool, batch, false, false, &h, &info)) return rc;
    Bf16Plan p;
    if (int rc = plan_bf16(pool, batch, h, q_heads / pool->kv_heads, flags, &p)) return rc;
    return p.quarters ? 16 : 32;
}

int ragc_batch_validate(const ragc_kv_pool* pool, const ragc_batch* batch, int32_t writes_new_tokens) {
    g_err[0] = 0;
    if (int rc = check_pool(pool)) return rc;
    BatchInfo info;
    HostMeta h;
    if (int rc = check_batch(pool, batch, true, true, &h, &info)) return rc;
    if (batch->num_reqs == 0) return RAGC_OK;
    return validate_batch(pool, batch, h, writes_new_tokens != 0);
}

int64_t ragc_prefill_attn_workspace(const ragc_kv_pool* pool, const ragc_batch* batch, int32_t q_heads, uint32_t flags) {
    g_err[0] = 0;
    if (int rc = check_pool(pool)) return rc;
    if (flags & ~kAttnFlags) return fail(RAGC_ERR_SHAPE, "unknown flags 0x%x", flags);
    if (q_heads <= 0 || q_heads % pool->kv_heads != 0)
        return fail(RAGC_ERR_SHAPE, "q_heads %d not a multiple of kv_heads %d", q_heads, pool->kv_heads);
    BatchInfo info;
    HostMeta h;
    if (int rc = check_batch(pool, batch, false, false, &h, &info)) return rc;
    if (pool->dtype != RAGC_DTYPE_BF16 || batch->num_reqs == 0 || info.total_new == 0) return 0;
    Bf16Plan plan;
    if (int rc = plan_bf16(pool, batch, h, q_heads / pool->kv_heads, flags, &plan)) return rc;
    return plan.workspace;
}

int ragc_prefill_attn(const ragc_kv_pool* pool, const ragc_batch* batch, const void* q, const void* k_new,
                      const void* v_new, void* out, int32_t q_heads, float softmax_scale, uint32_t flags,
                      void* workspace, size_t workspace_bytes, void* stream) {
    return prefill_attn_impl(pool, batch, q, k_new, v_new, out, q_heads, softmax_scale, flags, workspace, workspace_bytes,
                             false, stream);
}

int ragc_prefill_attn_static(const ragc_kv_pool* pool, const ragc_batch* batch, const void* q, const void* k_new,
                             const void* v_new, void* out, int32_t q_heads, float softmax_scale, uint32_t flags,
                             void* stream) {
    return prefill_attn_impl(pool, batch, q, k_new, v_new, out, q_heads, softmax_scale, flags, nullptr, 0, true, stream);
}

int ragc_kv_append(const ragc_kv_pool* pool, const ragc_batch* batch, const void* k_new, const void* v_new, void* stream) {
    g_err[0] = 0;
    if (int rc = check_pool(pool)) return rc;
    BatchInfo info;
    HostMeta h;
    if (int rc = check_batch(pool, batch, true, false, &h, &info)) return rc;
    if (batch->num_reqs == 0 || info.total_new == 0) return RAGC_OK;
    if (int rc = check_packed(batch, h)) return rc;
    if (!k_new || !v_new) return fail(RAGC_ERR_NULL, "k_new / v_new is NULL");
    if (!aligned16(k_new) || !aligned16(v_new)) return fail(RAGC_ERR_ALIGN, "k_new / v_new must be 16-byte aligned");
    const hipError_t e = ragc::launch_append(make_paged(pool, batch), pool->k, pool->v, k_new, v_new, (int32_t)info.total_new,
                                             esize_of(pool->dtype), static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return hip_fail(e, "append launch");
    return RAGC_OK;
}

int ragc_kv_gather(const ragc_kv_pool* pool, const ragc_batch* batch, int32_t req, int32_t length, void* k_out,
                   void* v_out, void* stream) {
    g_err[0] = 0;
    if (int rc = check_pool(pool)) return rc;
    if (!batch) return fail(RAGC_ERR_NULL, "batch is NULL");
    if (!batch->block_table) return fail(RAGC_ERR_NULL, "block_table is NULL");
    if (req < 0 || req >= batch->num_reqs) return fail(RAGC_ERR_RANGE, "req %d outside [0, %d)", req, batch->num_reqs);
    if (length < 0 || (int64_t)length > (int64_t)batch->table_stride * RAGC_BLOCK_SIZE)
        return fail(RAGC_ERR_RANGE, "length %d exceeds table capacity %lld", length, (long long)batch->table_stride * RAGC_BLOCK_SIZE);
    if (batch->h_block_table) {
        const int32_t* row = batch->h_block_table + (int64_t)req * batch->table_stride;
        for (int i = 0; i < (length + RAGC_BLOCK_SIZE - 1) / RAGC_BLOCK_SIZE; ++i)
            if (row[i] < 0 || row[i] >= pool->num_blocks)
                return fail(RAGC_ERR_RANGE, "block_table[%d] = %d outside [0, %d)", i, row[i], pool->num_blocks);
    }
    if (length == 0) return RAGC_OK;
    if (!k_out || !v_out) return fail(RAGC_ERR_NULL, "k_out / v_out is NULL");
    if (!aligned16(k_out) || !aligned16(v_out)) return fail(RAGC_ERR_ALIGN, "k_out / v_out must be 16-byte aligned");
    const hipError_t e = ragc::launch_gather(make_paged(pool, batch), req, length, k_out, v_out, esize_of(pool->dtype),
                                             static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return hip_fail(e, "gather launch");
    return RAGC_OK;
}

int ragc_kv_swap(const ragc_kv_pool* pool, void* host_k, void* host_v, int64_t host_block_stride_elems,
                 int32_t num_host_slots, const int32_t* dev_block_ids, const int32_t* host_slots, int32_t n,
                 int32_t direction, uint32_t flags, void* stream) {
    g_err[0] = 0;
    if (int rc = check_pool(pool)) return rc;
    if (!host_k || !host_v) return fail(RAGC_ERR_NULL, "host_k / host_v is NULL");
    if (n < 0) return fail(RAGC_ERR_RANGE, "n %d", n);
    if (direction != RAGC_SWAP_TO_DEVICE && direction != RAGC_SWAP_TO_HOST) return fail(RAGC_ERR_SHAPE, "direction %d", direction);
    if (flags > RAGC_SWAP_KERNEL) return fail(RAGC_ERR_SHAPE, "unknown swap flags 0x%x", flags);
    const int es = esize_of(pool->dtype);
    const int64_t plane_elems = (int64_t)pool->kv_heads * RAGC_BLOCK_SIZE * pool->head_dim;
    if (host_block_stride_elems < plane_elems)
        return fail(RAGC_ERR_SHAPE, "host_block_stride_elems %lld < %lld", (long long)host_block_stride_elems, (long long)plane_elems);
    if (!aligned16(host_k) || !aligned16(host_v) || (host_block_stride_elems * es) % 16 != 0)
        return fail(RAGC_ERR_ALIGN, "host planes and stride must be 16-byte aligned");
    if (num_host_slots <= 0) return fail(RAGC_ERR_SHAPE, "num_host_slots %d", num_host_slots);
    if (n == 0) return RAGC_OK;
    if (!dev_block_ids || !host_slots) return fail(RAGC_ERR_NULL, "dev_block_ids / host_slots is NULL");
    for (int i = 0; i < n; ++i) {
        if (dev_block_ids[i] < 0 || dev_block_ids[i] >= pool->num_blocks)
            return fail(RAGC_ERR_RANGE, "dev_block_ids[%d] = %d outside [0, %d)", i, dev_block_ids[i], pool->num_blocks);
        if (host_slots[i] < 0 || host_slots[i] >= num_host_slots)
            return fail(RAGC_ERR_RANGE, "host_slots[%d] = %d outside [0, %d)", i, host_slots[i], num_host_slots);
    }
    {  // two pairs must not write the same destination
        std::vector<int32_t> dst(direction == RAGC_SWAP_TO_DEVICE ? dev_block_ids : host_slots,
                                 (direction == RAGC_SWAP_TO_DEVICE ? dev_block_ids : host_slots) + n);
        std::sort(dst.begin(), dst.end());
        if (std::adjacent_find(dst.begin(), dst.end()) != dst.end())
            return fail(RAGC_ERR_RANGE, "two pairs write the same destination block");
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t plane_bytes = plane_elems * es;
    const int64_t dev_stride = pool->block_stride_elems * es;
    const int64_t host_stride = host_block_stride_elems * es;
    const bool to_dev = direction == RAGC_SWAP_TO_DEVICE;

    if (flags == RAGC_SWAP_MEMCPY) {
        // one copy per plane and run of pairs that are adjacent on both sides
        const bool dense = dev_stride == plane_bytes && host_stride == plane_bytes;
        int i = 0;
        while (i < n) {
            int j = i + 1;
            while (dense && j < n && dev_block_ids[j] == dev_block_ids[j - 1] + 1 && host_slots[j] == host_slots[j - 1] + 1) ++j;
            const size_t bytes = (size_t)(j - i) * plane_bytes;
            for (int plane = 0; plane < 2; ++plane) {
                char* d = static_cast<char*>(plane ? pool->v : pool->k) + (int64_t)dev_block_ids[i] * dev_stride;
                char* h = static_cast<char*>(plane ? host_v : host_k) + (int64_t)host_slots[i] * host_stride;
                const hipError_t e = to_dev ? hipMemcpyAsync(d, h, bytes, hipMemcpyHostToDevice, s)
                                            : hipMemcpyAsync(h, d, bytes, hipMemcpyDeviceToHost, s);
                if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");
            }
            i = j;
        }
        return RAGC_OK;
    }

    // copy kernel over the host-mapped pinned pool
    void *hk_dev = nullptr, *hv_dev = nullptr;
    hipError_t e = hipHostGetDevicePointer(&hk_dev, host_k, 0);
    if (e != hipSuccess) return hip_fail(e, "host_k is not pinned, device-mapped memory (hipHostGetDevicePointer)");
    e = hipHostGetDevicePointer(&hv_dev, host_v, 0);
    if (e != hipSuccess) return hip_fail(e, "host_v is not pinned, device-mapped memory (hipHostGetDevicePointer)");
    for (int i = 0; i < n; i += ragc::kSwapPairsPerLaunch) {
        const int cnt = std::min(ragc::kSwapPairsPerLaunch, n - i);
        ragc::SwapPairs pairs{};
        std::memcpy(pairs.dev, dev_block_ids + i, sizeof(int32_t) * cnt);
        std::memcpy(pairs.slot, host_slots + i, sizeof(int32_t) * cnt);
        e = ragc::launch_swap(static_cast<char*>(pool->k), static_cast<char*>(pool->v), dev_stride,
                              static_cast<char*>(hk_dev), static_cast<char*>(hv_dev), host_stride, plane_bytes, pairs, cnt,
                              to_dev ? 1 : 0, s);
        if (e != hipSuccess) return hip_fail(e, "swap kernel launch");
    }
    return RAGC_OK;
}

}  // extern "C"
