// How an attention workgroup finds its work (gfx950 device code, shared by the bf16 and fp32 kernels).
#pragma once
#include "ragc_internal.h"

namespace ragc {
namespace {

// Consecutive workgroup ids go round-robin over the 8 XCDs, each with an L2 of its own, so the kv head
// is taken from the low bits: all row tiles of one (request, kv head) stream share an L2.
__device__ __forceinline__ void split_block_id(int id, int kv_heads, int* g, int* entry) {
    if ((kv_heads & 7) == 0) {
        const int x = id & 7, j = id >> 3, hpx = kv_heads >> 3;
        *g = x + 8 * (j % hpx);
        *entry = j / hpx;
    } else {
        *g = id % kv_heads;
        *entry = id / kv_heads;
    }
}

struct WorkItem {
    int req, tile;  // request of the batch, row tile of the request
    int prefix, new_len, new_start;
};

// The request whose run of entries holds `entry`, and which of its row tiles that is (longest key range
// first).  Every lane fetches one request of the list and a ballot picks the right one: one trip to the
// kernel arguments, whatever the number of requests.
__device__ __forceinline__ WorkItem find_item(const AttnWork& wk, int entry, int group, int rows_per_tile, int lane) {
    int at = 0;
    while (at + 64 < wk.n_reqs && wk.req[at + 64].first <= entry) at += 64;
    const AttnReq rq = wk.req[at + lane];  // the list is padded to a multiple of 64
    const int id = wk.id[at + lane];
    const uint64_t below = __builtin_amdgcn_ballot_w64(at + lane < wk.n_reqs && rq.first <= entry);
    const int src = 63 - __builtin_clzll(below);
    WorkItem it;
    it.req = __builtin_amdgcn_readlane(id, src);
    it.prefix = __builtin_amdgcn_readlane(rq.prefix_len, src);
    it.new_len = __builtin_amdgcn_readlane(rq.new_len, src);
    it.new_start = __builtin_amdgcn_readlane(rq.new_start, src);
    const int tiles = (int)(((long long)it.new_len * group + rows_per_tile - 1) / rows_per_tile);
    it.tile = tiles - 1 - (entry - __builtin_amdgcn_readlane(rq.first, src));
    return it;
}

}  // namespace
}  // namespace ragc
