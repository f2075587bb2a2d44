// How an attention workgroup finds its work (gfx950 device code, shared by the bf16 and fp32 kernels).
#pragma once
#include "ragc_internal.h"

namespace ragc {
namespace {

// Everything a workgroup reads from the kernel arguments before it knows its work item, asked for at once: a
// launch's arguments are in no cache when it starts, and a first use here and there would cost a trip to memory each.
template <int REQS>
__device__ __forceinline__ void touch_args(const AttnLaunch& a, const AttnWorkN<REQS>& wk) {
    int touched = (int)(uintptr_t)a.pool_k | a.kv_heads | wk.first[0];
#pragma unroll
    for (int i = 0; i < kAttnReqStep; i += 64 / (int)sizeof(AttnReq)) touched |= wk.req[i].id;
    asm volatile("" ::"s"(touched));
}

// Consecutive workgroup ids go round-robin over the 8 XCDs, each with an L2 of its own, so the kv head
// is taken from the low bits: all row tiles of one (request, kv head) stream share an L2.
__device__ __forceinline__ void split_block_id(const AttnLaunch& a, int id, int* g, int* entry) {
    const int x = id & ((1 << a.head_shift) - 1), j = id >> a.head_shift;
    *entry = a.head_magic ? (int)__umulhi((uint32_t)j, a.head_magic) : j;
    *g = x + ((j - *entry * (int)a.head_div) << a.head_shift);
}

struct WorkItem {
    int req, tile;  // request of the batch, row tile of the request
    int prefix, new_len, new_start;
};

// The request whose run of items holds `item`, and which of its row tiles that is (longest key range first).
// Up to 16 requests by scalar compares, above one request per lane and a ballot (one trip to the arguments).
template <int REQS>
__device__ __forceinline__ WorkItem find_item(const AttnWorkN<REQS>& wk, int item, int group, int rows_per_tile) {
    WorkItem it;
    int first;
    if (REQS <= kAttnReqStep || wk.n_reqs <= kAttnReqStep) {
        // the last request whose first item is not above `item`, by halving; unused entries hold INT_MAX
        int f[kAttnReqStep], r = 0;
#pragma unroll
        for (int i = 0; i < kAttnReqStep; ++i) f[i] = wk.first[i];
#pragma unroll
        for (int half = kAttnReqStep / 2; half > 0; half /= 2) {
            const bool upper = f[half] <= item;
            r = upper ? r + half : r;
#pragma unroll
            for (int i = 0; i < half; ++i) f[i] = upper ? f[i + half] : f[i];
        }
        const AttnReq rq = wk.req[r];
        first = f[0];
        it = {rq.id, 0, rq.prefix_len, rq.new_len, rq.new_start};
    } else {
        const int lane = threadIdx.x & 63;
        int at = 0;
        while (at + 64 < wk.n_reqs && wk.first[at + 64] <= item) at += 64;
        const int lane_first = wk.first[at + lane];
        const AttnReq rq = wk.req[at + lane];  // the arrays are a multiple of 64 long
        const uint64_t below = __builtin_amdgcn_ballot_w64(at + lane < wk.n_reqs && lane_first <= item);
        const int src = 63 - __builtin_clzll(below);
        first = __builtin_amdgcn_readlane(lane_first, src);
        it = {__builtin_amdgcn_readlane(rq.id, src), 0, __builtin_amdgcn_readlane(rq.prefix_len, src),
              __builtin_amdgcn_readlane(rq.new_len, src), __builtin_amdgcn_readlane(rq.new_start, src)};
    }
    const int tiles = (int)(((long long)it.new_len * group + rows_per_tile - 1) / rows_per_tile);
    it.tile = tiles - 1 - (item - first);
    return it;
}

}  // namespace
}  // namespace ragc
