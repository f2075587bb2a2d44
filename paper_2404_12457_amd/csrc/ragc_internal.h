// Internal launch interface between the C-ABI front end (ragc_api.cpp) and the
// gfx950 kernels.  Not installed; the public contract is include/ragc.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ragc {

constexpr int kBlock = 16;  // tokens per paged block

// Records the text that ragc_last_error() returns on this thread; returns `code`.
int set_error(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));

// Everything a device kernel needs to find the K/V of a batch.
struct PagedBatch {
    const void* pool_k;
    const void* pool_v;
    int64_t block_stride;  // elements between blocks of one plane
    const int32_t* prefix_len;
    const int32_t* new_len;
    const int32_t* new_start;
    const int32_t* block_table;
    int32_t table_stride;
    int32_t num_reqs;
    int32_t kv_heads;
    int32_t head_dim;
};

// What every workgroup of an attention launch needs besides its work item.
struct AttnLaunch {
    void* pool_k;
    void* pool_v;
    int64_t block_stride;  // elements between blocks of one plane
    const int32_t* block_table;
    const void* q;
    const void* k_new;
    const void* v_new;
    void* out;
    void* partial;  // workspace for the partial results of work items split along the keys (bf16 path)
    int32_t table_stride;
    int32_t kv_heads;
    int32_t head_dim;
    int32_t q_heads;
    int32_t group;         // q_heads / kv_heads
    uint32_t group_magic;  // ceil(2^32 / group), 0 for group 1: row / group by one multiply in the kernels
    float scale_log2e;     // softmax_scale * log2(e)
    int32_t fused_append;
    int32_t head_shift;    // workgroup id -> (kv head, entry), see split_block_id: 3 if kv_heads is a multiple of 8, else 0,
    uint32_t head_div;     // kv_heads >> head_shift,
    uint32_t head_magic;   // and ceil(2^32 / head_div), 0 for 1
};

// The requests of one attention launch, in the kernel arguments: request i of the list owns the work
// items [first, first of the next one), one per row tile, and carries its lengths, so a workgroup
// needs no device array before it can look up its first block ids.  With `splits` = S > 1 every item is
// S work entries in a row (entry e is copy e % S of item e / S), and entry e leaves its partial result in
// slot part_base + e of the workspace.
constexpr int kAttnMaxReqs = 192;
constexpr int kAttnReqStep = 16;             // unused entries of `first` up to the next multiple hold INT_MAX
constexpr int kAttnMaxWorkgroups = 1 << 22;  // of one launch: grid times workgroup size stays below 2^32 threads
struct AttnReq {
    int32_t prefix_len;
    int32_t new_len;
    int32_t new_start;
    int32_t id;  // which request of the batch
};
template <int REQS>
struct AttnWorkN {
    int32_t n_reqs;
    int32_t splits;
    int32_t part_base;
    int32_t entry0;  // first entry of this launch (one launch holds so many workgroups)
    int32_t first[REQS];
    AttnReq req[REQS];
};
using AttnWork = AttnWorkN<kAttnMaxReqs>;
// A launch of up to kAttnReqStep requests takes a list of just that size: 0.45 KB of kernel arguments instead of
// 4 KB, which the host writes in 3.5 us per launch instead of 4.2.
using AttnWorkShort = AttnWorkN<kAttnReqStep>;
inline AttnWorkShort short_list(const AttnWork& w) {
    AttnWorkShort s;
    s.n_reqs = w.n_reqs;
    s.splits = w.splits;
    s.part_base = w.part_base;
    s.entry0 = w.entry0;
    for (int i = 0; i < kAttnReqStep; ++i) {
        s.first[i] = w.first[i];
        s.req[i] = i < w.n_reqs ? w.req[i] : AttnReq{};
    }
    return s;
}

// fp32 path (attn_f32.hip): row tiles of 16 rows, or of 32 for the kernel that splits its operands
constexpr int kAttnF32Rows = 16;
constexpr int kAttnF32SplitRows = 32;
// rows: one of these; waves: 4 or 8 per workgroup
hipError_t launch_attn_f32(const AttnLaunch& a, const AttnWork& wk, int entries, int rows, int waves, hipStream_t s);

// bf16 path.  Large batches: row tiles of kAttnRowsPerItem rows (attn_bf16.hip).  Launches that cannot fill the chip
// with those: kAttnShortRows rows (attn_bf16_rows.hip), or either split along the keys.
constexpr int kAttnRowsPerItem = 128;
constexpr int kAttnShortRows = 32;
// bytes of one partial result of a key-split item: O [rows][D] fp32, then (max, sum) per row
inline int64_t attn_partial_bytes(int head_dim, int rows) { return (int64_t)rows * (head_dim + 2) * 4; }
constexpr int kAttnMaxSplits = 16;
enum AttnVariant {
    kAttnVariantOneGroup = 0,   // 4 waves per workgroup, two workgroups per CU
    kAttnVariantTwoGroups = 1,  // 8 waves per workgroup on alternating key tiles
    kAttnVariantCount = 2
};
// entries: items times wk.splits, from wk.entry0 on; split items are kAttnVariantOneGroup
// quarters: at head_dim 128, items not split, take the 16x16x32 products (a row in four lanes) instead of 32x32x16
hipError_t launch_attn_bf16(const AttnLaunch& a, const AttnWork& wk, int entries, int variant, bool quarters, hipStream_t s);
// waves: 4 or 8 per workgroup; split items have 8
hipError_t launch_attn_bf16_rows(const AttnLaunch& a, const AttnWork& wk, int entries, int waves, hipStream_t s);
// second pass after a launch of split items of `rows` rows: combines the partial results into `out`
hipError_t launch_attn_bf16_merge(const AttnLaunch& a, const AttnWork& wk, int entries, int rows, hipStream_t s);

hipError_t launch_append(const PagedBatch& b, void* pool_k, void* pool_v, const void* k_new, const void* v_new,
                         int32_t total_new, int esize, hipStream_t s);
hipError_t launch_gather(const PagedBatch& b, int32_t req, int32_t length, void* k_out, void* v_out, int esize,
                         hipStream_t s);

// Block copies between the device pool and a host-mapped pinned pool.  Pairs are
// passed by value in the kernel argument buffer, so no device staging is needed.
constexpr int kSwapPairsPerLaunch = 384;
struct SwapPairs {
    int32_t dev[kSwapPairsPerLaunch];
    int32_t slot[kSwapPairsPerLaunch];
};
hipError_t launch_swap(char* dev_k, char* dev_v, int64_t dev_block_bytes_stride, char* host_k, char* host_v,
                       int64_t host_block_bytes_stride, int64_t plane_block_bytes, const SwapPairs& pairs, int32_t n,
                       int to_device, hipStream_t s);

}  // namespace ragc
