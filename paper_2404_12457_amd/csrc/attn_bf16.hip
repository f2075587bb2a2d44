// bf16 prefix-cached paged prefill attention on gfx950 matrix cores.
//
// out[t,h,:] = softmax_j(scale * q[t,h,:].K_j) V_j over j = 0..prefix+i: the first
// `prefix` keys come from 16-token pool blocks through the request's block table
// (paper Sec. 5.1: K/V of cached documents lives in non-contiguous blocks referenced
// by tree nodes), the rest are the request's own fresh K/V (Sec. 3.2: only the
// request tokens are computed), and the same pass can store that fresh K/V into its
// paged slots (Sec. 4: tensors are cached after the first token).
//
// Mapping.  One work item = (request, kv head, 128 rows); a row is a (new token,
// q head of the group) pair, token-major, so the G q heads of a GQA group share
// every K/V tile and a tile's causal frontier stays narrow.  A wave owns 32 rows.
// Keys stream through LDS in tiles of 64 (four pool blocks): each wave copies one
// 16-token block of K and of V per tile straight from HBM into LDS
// (global_load_lds, 16 bytes per lane), one tile ahead of the math, into a ring of
// stages.  Rows are stored unpadded with their 16-byte chunks XOR-swizzled so that
// both the 16-byte K reads and the transposing V reads are bank-conflict free.
//
// NG wave groups of 4 waves work on the same 128 rows but on alternating key tiles
// (each with its own online-softmax state, merged through LDS at the end), so that a
// launch with few work items still puts 8 waves on a CU and one group's softmax
// overlaps the other's MFMAs.  With many work items NG = 1 and two workgroups share
// a CU instead.
//
// Launches too small to fill the chip with such items go to attn_bf16_rows_kernel, or are split along
// the keys ACROSS workgroups (SPLIT, NG = 1): every item then appears S times, each copy walks 1/S of
// the key tiles and leaves its unnormalised O and its (max, sum) per row in the caller's workspace,
// and attn_bf16_merge_kernel combines the S partial results of every row.
//
// The products are computed transposed so that a lane owns ONE query row:
//   S^T[key][row] = K . Q^T      A = K tile (LDS, 16-byte reads), B = Q (registers)
//   O^T[d][row]  += V^T . P^T    A = V tile read with the transposing LDS load,
//                                B = P^T, which is exactly the accumulator layout of
//                                S^T after conversion to bf16 -- no data movement.
// The row's reference exponent is only raised (and O, l rescaled) when a tile's probabilities
// against it sum to more than 2^8.
//
// What bounds it, and which product.  With every CU busy the power limit holds the clock at 1.5 to
// 2.1 GHz, and then a product's energy counts more than its cycles: on random operands a loop of
// v_mfma_f32_16x16x32_bf16 sustains 1852 TFLOP/s at 2.07 GHz where 32x32x16, which moves the
// accumulators through the registers twice as often per flop, sustains 1640 at 1.77.  Per cycle it is
// the slower one (16.5-17 instead of 16 in a loop), which shows while a launch is too short or too
// small for the limit to take hold.  So at head_dim 128 launches of 12000 keys (times 32 rows) per CU
// and more, 50 GFLOP in all, or of 1500 where there are three items per CU and more, take 16x16x32
// (KG = 4: two blocks of 16 rows per wave, a row in four lanes): on a warm card 4 x (4096 + 128) tokens
// of 64/8 heads 68.6 us with 32x32x16 and 66.6 with 16x16x32, eight of them 141.6 and 136, 16 x (256-4096 +
// 64-768) of 32/8 heads 293 and 289.5, four whole prompts of 2200-3500 245 and 240; ragged batches of two
// to three items per CU go either way, by up to 4 %.  Others take 32x32x16 (KG = 2: one block of 32 rows, a
// row in two lanes): below 12000 0.98 of the time (medians of 38 batches; 64/8 heads, 200-592 + 486 tokens
// 17.8 us against 18.5); with three items per CU 0.97-1.00 up to 1300 (1360 items of 9-37 tokens without a
// prefix 21.2 against 21.9), but 0.99-1.03 from 1500 to 12000 (1866 of 180-365 tokens 54.2 against 53.0).
// At head_dim 64, where a step has half the products for the same softmax, 320 items of 450-1900 keys
// take 21.5 us against 22.7, and only with the chip full of long items is it the other way round (2048
// of 4224 keys: 81 us against 78).
#include "attn_bf16_common.h"
#include "attn_work.h"

namespace ragc {
namespace {

constexpr int TM = kAttnRowsPerItem;  // rows per work item

template <int N, class F>
__device__ __forceinline__ void static_for(const F& f) {
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

__device__ __forceinline__ f32x16 product(bf16x8 a, bf16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4 product(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

template <int D, int NG, int KG, bool SPLIT, class Work>
__global__ __launch_bounds__(256 * NG, NG == 1 ? 2 : 1) void attn_bf16_kernel(AttnLaunch a, Work wk) {
    static_assert(!SPLIT || (NG == 1 && KG == 2), "copies of an item are one wave group each, with 32x32x16 products");
    constexpr int RING = 2;             // stages per wave group
    // Which product: v_mfma_f32_16x16x32_bf16 (KG = 4) or 32x32x16 (KG = 2).  A lane is row lane % BR and group lane / BR: KG
    // lanes per row, each with every KG-th run of four keys or columns.
    constexpr int BR = 64 / KG;         // rows, keys and columns of a product
    constexpr int CK = 8 * KG;          // its contraction
    constexpr int NE = 16 / (KG * KG / 4);  // accumulators per lane
    constexpr int NSUB = TN / BR;       // BR-key subtiles of a tile
    constexpr int RB = 32 / BR;         // BR-row blocks of a wave
    typedef __attribute__((ext_vector_type(NE))) float accv;
    constexpr int CPR = D / 8;          // 16-byte chunks per K/V row
    constexpr int ROWB = D * 2;         // bytes per row
    constexpr int PLANEB = TN * ROWB;   // one tile of K (or V)
    constexpr int STAGEB = 2 * PLANEB;
    constexpr int RPI = 64 / CPR;       // rows covered by one wave-wide 1 KiB DMA instruction
    constexpr int IPB = 16 / RPI;       // DMA instructions per 16-row block and plane
    constexpr int KSTEPS = D / CK;
    constexpr int PSTEPS = TN / CK;     // contraction steps of P.V
    constexpr int DB = D / BR;          // BR-column blocks of the output
    constexpr int NSTAGE = NG * RING;
    static_assert(NSTAGE * STAGEB <= 160 * 1024, "LDS");
    __shared__ __attribute__((aligned(1024))) char smem[NSTAGE * STAGEB];

    touch_args(a, wk);
    const int Hkv = a.kv_heads;
    int g, entry;
    split_block_id(a, blockIdx.x, &g, &entry);
    entry += wk.entry0;
    const int tid = threadIdx.x, lane = tid & 63, kg = lane / BR, lrow = lane % BR;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = NG == 1 ? 0 : w >> 2, wq = w & 3;
    const int S = SPLIT ? wk.splits : 1, sidx = SPLIT ? entry % S : 0;
    const WorkItem it = find_item(wk, SPLIT ? entry / S : entry, a.group, TM);
    const int tile = it.tile;

    const int G = a.group;
    // x / G for 0 <= x < 2^26 / G without an integer division (the host supplies ceil(2^32 / G), 0 for G = 1)
    const uint32_t g_magic = a.group_magic;
    auto div_g = [&](int x) { return g_magic ? (int)__umulhi((uint32_t)x, g_magic) : x; };
    const int N = it.new_len;
    const int rows_total = N * G;
    const int row0 = tile * TM;
    const int P = it.prefix;
    const int s0 = it.new_start;
    const int Hq = a.q_heads;

    const __bf16* __restrict__ q = static_cast<const __bf16*>(a.q);
    const __bf16* __restrict__ k_new = static_cast<const __bf16*>(a.k_new);
    const __bf16* __restrict__ v_new = static_cast<const __bf16*>(a.v_new);
    const __bf16* __restrict__ pool_k = static_cast<const __bf16*>(a.pool_k);
    const __bf16* __restrict__ pool_v = static_cast<const __bf16*>(a.pool_v);
    const int32_t* __restrict__ table = a.block_table + (long long)it.req * a.table_stride;

    const int last_row = min(row0 + TM, rows_total) - 1;
    const int kv_limit = P + div_g(last_row) + 1;  // keys [0, kv_limit) are visible to some row of the item
    const int ntiles_all = (kv_limit + TN - 1) / TN;
    // copy sidx of S takes tiles [t_lo, ntiles); more copies than tiles: nothing for some, but each of them leaves a state
    const int t_lo = ntiles_all * sidx / S, ntiles = ntiles_all * (sidx + 1) / S;
    const int nsteps = (ntiles - t_lo + NG - 1) / NG;  // group `grp` takes tile t_lo + step*NG + grp

    // ---- this lane's query row
    const int wrow0 = row0 + wq * 32;
    int my_vis[RB];  // keys [0, my_vis) are visible to row lrow of each block
    const __bf16* qp[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int my_row = min(wrow0 + rb * BR + lrow, rows_total - 1);  // rows past the end repeat the last one
        const int my_tok = div_g(my_row);
        my_vis[rb] = P + my_tok + 1;
        qp[rb] = q + ((long long)(s0 + my_tok) * Hq + g * G + (my_row - my_tok * G)) * D + kg * 8;
    }
    const bool wave_active = wrow0 < rows_total;
    const int wave_vis_min = P + div_g(wrow0) + 1;
    const int wave_vis_max = P + div_g(min(wrow0 + 31, rows_total - 1)) + 1;

    // Block ids are fetched 64 steps at a time, one per lane (entry of step blk_base+lane), and
    // handed out with a lane read: no memory load sits on the issue path of a step.  The first
    // window is requested before Q so that both round trips overlap; it also covers the blocks of
    // this item's new tokens, which warms the table lines the fused append reads at the end.
    const int nblk_item = (kv_limit + 15) >> 4;
    int blk_base = 0;
    int blk_vec;
    {
        const int e = (min(t_lo + lane * NG + grp, max(ntiles - 1, 0)) * TN >> 4) + wq;
        blk_vec = e < nblk_item ? table[e] : 0;
    }
    bf16x8 qreg[RB][KSTEPS];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) qreg[rb][ks] = *reinterpret_cast<const bf16x8*>(qp[rb] + ks * CK);
    // Every ordinary load above completes here, before the DMA ring starts counting.  The
    // empty asm statements make the compiler itself wait for these registers now; otherwise it
    // would place its vmcnt waits at their first use inside the loop and drain the ring there.
    asm volatile("" ::"v"(blk_vec));
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) asm volatile("" ::"v"(qreg[rb][ks]));
    wait_vmcnt<0>();

    // ---- DMA: wave (grp, wq) copies block wq (16 keys) of tile step*NG+grp, K and V planes.
    // Lane i of DMA instruction c brings row RPI*c + i/CPR of the block, 16-byte chunk
    // (i%CPR) ^ swz(row): the swizzle is applied on the global side, LDS is written linearly.
    // Byte offsets of this lane's chunks inside the source, less what the instruction's own offset adds: inside a pool
    // block, or (from the first fresh block on) inside a run of fresh rows.
    uint32_t loff[IPB];
    auto set_loff = [&](int row_stride) {
#pragma unroll
        for (int c = 0; c < IPB; ++c) {
            const int row16 = RPI * c + lane / CPR;
            const int chunk = (lane % CPR) ^ swz<D, KG>(row16);
            loff[c] = (row16 * row_stride + chunk * 8) * 2 - c * 1024;
        }
    };
    const uint32_t smem_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    // The copy of one step is prepared (addresses) right after the barrier and its DMA
    // instructions are then slipped between the MFMAs of S^T = K.Q^T, where their issue cost
    // hides under the matrix pipe; `flush` issues whatever is still pending at once.
    int pend = 0;              // 1: a fast-path copy (uniform base + per-lane constant) waits to be issued
    uint64_t pend_kb = 0, pend_vb = 0;
    uint32_t pend_dst = 0;
    // copy instructions 2 i and 2 i + 1 of the 2 IPB of a step, K first, then V
    auto emit = [&](auto i_c) {
        constexpr int I = 2 * decltype(i_c)::value, C = I % IPB;
        dma_runs<2, C * 1024>(I < IPB ? pend_kb : pend_vb, loff + C, I < IPB ? pend_dst : pend_dst + PLANEB);
    };
    auto flush = [&]() {
        if (pend) {
            static_for<IPB>(emit);
            pend = 0;
        }
    };
    // All of `prepare` stands between the barrier and the first product of a step.  For a block that is cached as a whole -- most
    // of them -- it is one branch, laid out as the way straight ahead, a lane read and a few scalar sums: the base of the head is
    // made once (made anew in 64 bits at each step: 8 x (4096 + 128) tokens of 64/8 heads 137.6 us against 135.1).  Counting these
    // steps beforehand, three scalar instructions less in each, is no faster (137.3), and what it takes before the first copy and
    // in scalar registers, some of them spilled, costs prompts of one tile 1-3 % (512 items of head_dim 64 9.07 us against 8.83,
    // 400 of 9-11 tokens, 32/8 heads of 128, 13.66 against 13.39).
    const uint64_t block_bytes = (uint64_t)a.block_stride * 2;
    const uint64_t head_k = uniform_u64(pool_k + (long long)g * kBlock * D), head_v = uniform_u64(pool_v + (long long)g * kBlock * D);
    const uint32_t copy_dst = smem_addr + grp * RING * STAGEB + wq * 16 * ROWB;
    set_loff(D);
    bool loff_fresh = false;
    auto prepare = [&](int step) {
        if (step - blk_base >= 64) {
            blk_base = step;
            const int e = (min(t_lo + (step + lane) * NG + grp, ntiles - 1) * TN >> 4) + wq;
            blk_vec = e < nblk_item ? table[e] : 0;
            asm volatile("" ::"v"(blk_vec));  // the compiler's wait for this load stays inside the branch
        }
        const int blk = __builtin_amdgcn_readlane(blk_vec, step - blk_base);
        const int tg = min(t_lo + step * NG + grp, ntiles - 1);  // a group without a tile re-reads the last one (same count of loads)
        const int kbase = tg * TN + wq * 16;
        const uint32_t dst = copy_dst + step % RING * STAGEB;
        if (__builtin_expect(kbase + 16 <= P, 1)) {
            // one pool block, uniform base + per-lane constant
            const uint64_t boff = (uint32_t)blk * block_bytes;
            pend_kb = head_k + boff;
            pend_vb = head_v + boff;
            pend_dst = dst;
            pend = 1;
        } else if (kbase >= P && kbase + 16 <= kv_limit) {
            // 16 fresh rows, all inside the horizon
            const long long boff = (((long long)(s0 + kbase - P)) * Hkv + g) * D * 2;
            pend_kb = uniform_u64(reinterpret_cast<const char*>(k_new) + boff);
            pend_vb = uniform_u64(reinterpret_cast<const char*>(v_new) + boff);
            pend_dst = dst;
            if (!loff_fresh) {  // no pool block follows
                loff_fresh = true;
                set_loff(Hkv * D);
            }
            pend = 1;
        } else {
            // the block straddles the prefix end or the horizon: choose the source per row, issue
            // now; rows past the horizon re-read the last visible one (they are masked later)
#pragma unroll
            for (int c = 0; c < IPB; ++c) {
                const int row16 = RPI * c + lane / CPR;
                const int chunk = (lane % CPR) ^ swz<D, KG>(row16);
                const int kj = kbase + row16;
                long long off;
                if (kj < P) {
                    off = (long long)blk * a.block_stride + ((long long)g * kBlock + row16) * D + chunk * 8;
                } else {
                    const int kn = min(kj, kv_limit - 1) - P;
                    off = ((long long)(s0 + kn) * Hkv + g) * D + chunk * 8;
                }
                const __bf16* ksrc = (kj < P ? pool_k : k_new) + off;
                const __bf16* vsrc = (kj < P ? pool_v : v_new) + off;
                dma_16B_per_lane(ksrc, dst + RPI * c * ROWB);
                dma_16B_per_lane(vsrc, dst + RPI * c * ROWB + PLANEB);
            }
            pend = 0;
        }
    };

    // ---- per-lane LDS read offsets (bytes); the stage and sub-tile parts are immediates
    typedef __attribute__((address_space(3))) char lds_char;
    lds_char* const lds0 = (lds_char*)smem;
    const int grp_off = grp * RING * STAGEB;  // folded into the per-lane offsets below
    // K, A operand of S^T: row sub*BR+lrow, chunk KG*ks+kg
    int koff[KSTEPS];
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
        koff[ks] = grp_off + lrow * ROWB + (((KG * ks + kg) ^ swz<D, KG>(lrow)) << 4);
        asm volatile("" : "+v"(koff[ks]));  // keep it one register: address = this + immediate
    }
    // V, A operand of O^T (transposing reads): rows step*CK + h2*4*KG + 4*kg + (lane%16)/4, 8 bytes at element
    // db*BR + (second 16 lanes of 32: 16) + 4*(lane%4).  Rows 16 apart are swizzled alike: one offset for both reads.
    constexpr int NH = KG == 2 ? 2 : 1;
    int voff[NH][DB];
#pragma unroll
    for (int h2 = 0; h2 < NH; ++h2)
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const int row = h2 * 4 * KG + 4 * kg + ((lane & 15) >> 2);
            const int elem = db * BR + (lane % BR / 16) * 16 + 4 * (lane & 3);
            voff[h2][db] = grp_off + row * ROWB + (((elem >> 3) ^ swz<D, KG>(row)) << 4) + (elem & 7) * 2;
            asm volatile("" : "+v"(voff[h2][db]));
        }

    accv oacc[DB][RB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) oacc[db][rb] = accv(0.f);
    float m_run[RB], l_run[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        m_run[rb] = -INFINITY;  // reference exponent of O and l (log2 domain): a lane's probabilities of a tile sum to at most 2^8
        l_run[rb] = 0.f;        // this lane's partial of the running sum
    }
    const float c = a.scale_log2e;

    // one step with the ring slot as a compile-time constant
    auto do_step = [&](int step, auto slot_c) {
        constexpr int SLOT = decltype(slot_c)::value;
        wait_vmcnt<0>();  // the copies of this step have landed
        block_barrier();  // every wave's part is in LDS, and every wave is done with the previous step
        if (step + 1 < nsteps) prepare(step + 1);

        const int tg = t_lo + step * NG + grp;
        const int base = tg * TN;  // first key this wave looks at
        if (!wave_active || tg >= ntiles || base >= wave_vis_max) {
            flush();
            return;
        }
        lds_char* const kst = lds0 + SLOT * STAGEB;
        lds_char* const vst = kst + PLANEB;

        // S^T = K Q^T
        accv sacc[NSUB][RB];
#pragma unroll
        for (int sub = 0; sub < NSUB; ++sub)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) sacc[sub][rb] = accv(0.f);
        // Two K operands at a time, read two such groups ahead (a group is 64 cycles of products, about half the LDS latency).
        constexpr int GROUPS = KSTEPS * NSUB / 2;
        static_assert(GROUPS % 2 == 0, "the copies, which may be skipped by a branch, stand behind even groups only: never "
                                       "between the last products and the first read of their results");
        bf16x8 kbuf[3][2];
        auto read_k = [&](auto g_c) {
            constexpr int GI = decltype(g_c)::value;
#pragma unroll
            for (int x = 0; x < 2; ++x)
                kbuf[GI % 3][x] = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(kst + (2 * GI + x) % NSUB * BR * ROWB + koff[(2 * GI + x) / NSUB]);
        };
        read_k(std::integral_constant<int, 0>{});
        read_k(std::integral_constant<int, 1>{});
        static_for<GROUPS>([&](auto g_c) {
            constexpr int GI = decltype(g_c)::value;
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (GI + 2 < GROUPS) read_k(std::integral_constant<int, GI + 2>{});
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    accv& s = sacc[(2 * GI + x) % NSUB][rb];
                    s = product(kbuf[GI % 3][x], qreg[rb][(2 * GI + x) / NSUB], s);
                }
            // Two copy instructions behind every other group: 8 waves of a CU that issue theirs in one burst after the
            // barrier queue for the address unit (all behind the first half: 16 x (256-4096 + 64-768) tokens, 32/8
            // heads 300 us against 296, 12 x (1000-2000 + 60-200) 77.6 against 75.8).
            if constexpr (GI % 2 == 0) {
                if (pend) emit(std::integral_constant<int, GI / 2>{});
            }
        });
        bf16x8 vbuf[3][2];
        auto read_v = [&](auto g_c) {
            constexpr int GI = decltype(g_c)::value;
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                constexpr int STEP = 2 * GI / DB;
                const int db = (2 * GI + x) % DB;
                lds_char* const vb = vst + STEP * CK * ROWB;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(vb + voff[0][db]));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(vb + (NH - 1 ? 0 : 4 * KG * ROWB) + voff[NH - 1][db]));
                vbuf[GI % 3][x] = __builtin_shufflevector(__builtin_bit_cast(bf16x4, lo), __builtin_bit_cast(bf16x4, hi), 0, 1, 2, 3, 4, 5, 6, 7);
            }
        };
        read_v(std::integral_constant<int, 0>{});
        read_v(std::integral_constant<int, 1>{});
        pend = 0;
        // causal frontier / end of sequence: only tiles that reach past the first row's horizon
        if (base + TN > wave_vis_min) {
#pragma unroll
            for (int sub = 0; sub < NSUB; ++sub)
#pragma unroll
                for (int i = 0; i < NE; ++i) {
                    const int kidx = base + sub * BR + (i >> 2) * (4 * KG) + kg * 4 + (i & 3);
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
                        if (kidx >= my_vis[rb]) sacc[sub][rb][i] = -INFINITY;
                }
        }
        // Online softmax, one row per KG lanes, without a maximum: the probabilities are taken against
        // the row's reference exponent as it stands, and only where a lane's sum of them says that a score may be 2^8 above
        // it (or that the row has no reference yet: 2^inf, or NaN where every key is masked) is the maximum looked up, the
        // reference raised and O, l rescaled.  Against a maximum per tile this takes 22 vector instructions and the trip
        // maximum -> ballot -> branch -> exponentials out of a step: 24 requests at head_dim 64 73.5 -> 70.4 us, 12 x
        // (1000-2000 + 60-200) tokens at 128 79.3 -> 77.2, others equal or better.  The first step looks the maximum up at
        // once: weighing twice there cost 4 % on calls of one or two tiles.  One check per 32 keys instead of 64: 5 % more
        // on the first of these, 9 % less on batches with one item per CU.
        // The row sum is taken over the bf16-rounded probabilities, the same weights the PV product uses, so that the
        // rounding of P cancels between numerator and denominator.
        bf16x8 pb[RB][PSTEPS];  // the scores' order of keys, which the V reads follow
        float psum[RB];
        auto weigh = [&](int rb, float m_sub) {
            psum[rb] = 0.f;
#pragma unroll
            for (int sub = 0; sub < NSUB; ++sub)
#pragma unroll
                for (int i = 0; i < NE; i += 2) {
                    const int e = sub * NE + i;
                    const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[sub][rb][i], c, -m_sub));
                    const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[sub][rb][i + 1], c, -m_sub));
                    const bf16x2 pp = {(__bf16)p0, (__bf16)p1};
                    psum[rb] = __builtin_amdgcn_fdot2_f32_bf16(pp, kOnes2, psum[rb], false);
                    pb[rb][e >> 3][e & 7] = pp[0];
                    pb[rb][e >> 3][(e & 7) + 1] = pp[1];
                }
        };
        bool raise_any = step == 0;  // there the rows have no reference yet, as a rule
        if (!raise_any) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) weigh(rb, m_run[rb]);
            raise_any = __builtin_amdgcn_ballot_w64(!(psum[0] <= kRaiseSum) || !(psum[RB - 1] <= kRaiseSum)) != 0;
        }
        if (raise_any) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                float mx = sacc[0][rb][0];
#pragma unroll
                for (int sub = 0; sub < NSUB; ++sub)
#pragma unroll
                    for (int i = 0; i < NE; ++i) mx = fmaxf(mx, sacc[sub][rb][i]);
                mx = fmaxf(mx, other_half(mx));
                if (KG == 4) mx = fmaxf(mx, other_quarter(mx));
                mx *= c;
                const bool raise = mx > m_run[rb];
                const float alpha = raise ? __builtin_amdgcn_exp2f(m_run[rb] - mx) : 1.f;  // 0 where the row has no reference yet
                m_run[rb] = raise ? mx : m_run[rb];
                l_run[rb] *= alpha;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int i = 0; i < NE; ++i) oacc[db][rb][i] *= alpha;
                weigh(rb, m_run[rb] == -INFINITY ? 0.f : m_run[rb]);  // still no visible key: exp2(-inf - 0) = 0
            }
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) l_run[rb] += psum[rb];

        // O^T += V^T P^T, two column blocks at a time over CK keys, so that a product waits for none of those just before it
        constexpr int VGROUPS = PSTEPS * DB / 2;
        static_for<VGROUPS>([&](auto g_c) {
            constexpr int GI = decltype(g_c)::value;
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (GI + 2 < VGROUPS) read_v(std::integral_constant<int, GI + 2>{});
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    accv& o = oacc[(2 * GI + x) % DB][rb];
                    o = product(vbuf[GI % 3][x], pb[rb][2 * GI / DB], o);
                }
        });
    };

    if (!SPLIT || nsteps > 0) {
        prepare(0);
        flush();
    }
    for (int step0 = 0; step0 < nsteps; step0 += RING) {
        do_step(step0, std::integral_constant<int, 0>{});
        if (step0 + 1 < nsteps) do_step(step0 + 1, std::integral_constant<int, 1>{});
    }

    // ---- fused append (after the key loop: nothing waits for it, and the fresh rows are L2-hot
    // because the loop has just read them as keys; requested up front, next to Q, the rows cost 1-4 %
    // on the prefill configurations and gain 1-2 % on decode steps).  This work item (its last copy) owns the tokens
    // whose first row (head 0 of the group) it holds; 16-byte chunks, four per thread in flight.
    if (a.fused_append && sidx == S - 1) {
        const int tok_lo = div_g(row0 + G - 1);
        const int tok_hi = min(N - 1, div_g(row0 + TM - 1));
        __bf16* wk = static_cast<__bf16*>(a.pool_k);
        __bf16* wv = static_cast<__bf16*>(a.pool_v);
        const int n = (tok_hi - tok_lo + 1) * CPR;
        constexpr int UNR = 4;
        for (int i0 = tid; i0 < n; i0 += (256 * NG) * UNR) {
            int blk[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const int idx = min(i0 + u * (256 * NG), n - 1);
                blk[u] = table[(P + tok_lo + idx / CPR) >> 4];
            }
            u32x4 kk[UNR], vv[UNR];
            long long dst[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const int idx = min(i0 + u * (256 * NG), n - 1);
                const int tok = tok_lo + idx / CPR, ch = idx % CPR;
                const int pos = P + tok;
                const long long src = ((long long)(s0 + tok) * Hkv + g) * D + ch * 8;
                dst[u] = (long long)blk[u] * a.block_stride + ((long long)g * kBlock + (pos & 15)) * D + ch * 8;
                kk[u] = *reinterpret_cast<const u32x4*>(k_new + src);
                vv[u] = *reinterpret_cast<const u32x4*>(v_new + src);
            }
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                if (i0 + u * (256 * NG) < n) {
                    *reinterpret_cast<u32x4*>(wk + dst[u]) = kk[u];
                    *reinterpret_cast<u32x4*>(wv + dst[u]) = vv[u];
                }
            }
        }
    }

    // ---- merge the wave groups through LDS (the DMA ring is idle now)
    constexpr int OC = NE / 4;  // 16-byte chunks of an accumulator
    constexpr int WSTRIDE = (DB * RB * OC * 4 + 4) * 64;  // floats per wave in the merge area: [DB*RB*OC + 1 chunks][64 lanes][4]
    auto ochunk = [&](int db, int rb, int i4) { return f32x4{oacc[db][rb][i4 * 4], oacc[db][rb][i4 * 4 + 1], oacc[db][rb][i4 * 4 + 2], oacc[db][rb][i4 * 4 + 3]}; };
    if (NG > 1) {
        typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
        lds_f32x4* const xw = reinterpret_cast<lds_f32x4*>(lds0 + wq * (WSTRIDE * 4)) + lane;
        block_barrier();
        if (grp == 1) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int i4 = 0; i4 < OC; ++i4) xw[((db * RB + rb) * OC + i4) * 64] = ochunk(db, rb, i4);
            const f32x4 ml = {m_run[0], l_run[0], m_run[RB - 1], l_run[RB - 1]};
            xw[DB * RB * OC * 64] = ml;
        }
        block_barrier();
        if (grp == 1) return;
        if (wave_active) {
            const f32x4 ml = xw[DB * RB * OC * 64];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const float m1 = ml[2 * rb], l1 = ml[2 * rb + 1];
                // a group may have seen no visible key of a row: weight 0 (which lets NaN through)
                const float m = fmaxf(m_run[rb], m1);
                const float s0f = m_run[rb] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run[rb] - m);
                const float s1f = m1 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m1 - m);
                m_run[rb] = m;
                l_run[rb] = l_run[rb] * s0f + l1 * s1f;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int i4 = 0; i4 < OC; ++i4) {
                        const f32x4 v = xw[((db * RB + rb) * OC + i4) * 64];
#pragma unroll
                        for (int e = 0; e < 4; ++e) oacc[db][rb][i4 * 4 + e] = oacc[db][rb][i4 * 4 + e] * s0f + v[e] * s1f;
                    }
            }
        }
    } else {
        block_barrier();  // every wave is done with the ring: its memory is reused below
    }

    // ---- normalise and store.  A lane holds 4 consecutive d of ONE row per (dt, i/4), so a direct
    // store would touch 32 rows with 16 bytes each per instruction; instead the wave turns its 32
    // rows around in a private LDS patch (rows padded by 16 bytes) and stores whole rows, 16 bytes
    // per lane.  With two groups the patch is the wave's own merge area, which only it reads.
    if (!wave_active) return;
    constexpr int OROWB = ROWB + 16;
    static_assert(32 * OROWB <= WSTRIDE * 4, "output patch fits the merge area");
    lds_char* const patch = lds0 + wq * (NG > 1 ? WSTRIDE * 4 : 32 * OROWB);
    float l_tot[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        l_tot[rb] = l_run[rb] + other_half(l_run[rb]);
        if (KG == 4) l_tot[rb] += other_quarter(l_tot[rb]);
    }
    if (SPLIT) {
        // one of S copies: O (unnormalised, fp32), max and sum of every row go to the workspace, [TM][D] floats of O, then
        // [TM][2] floats (max, sum).  Same turn through LDS as below, in two passes of D/2 floats per row.
        float* const part = static_cast<float*>(a.partial) + ((long long)(wk.part_base + entry) * Hkv + g) * (TM * (D + 2));
        if (kg == 0) *reinterpret_cast<float2*>(part + TM * D + (wq * 32 + lrow) * 2) = float2{m_run[0], l_tot[0]};
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
            for (int dbl = 0; dbl < DB / 2; ++dbl)
#pragma unroll
                for (int i4 = 0; i4 < OC; ++i4)
                    *reinterpret_cast<__attribute__((address_space(3))) f32x4*>(patch + lrow * OROWB + (dbl * BR + i4 * 4 * KG + kg * 4) * 4) =
                        ochunk(pass * (DB / 2) + dbl, 0, i4);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int p = 0; p < 32 / RPI; ++p) {
                const int rr = p * RPI + lane / CPR;
                const f32x4 v = *reinterpret_cast<const __attribute__((address_space(3))) f32x4*>(patch + rr * OROWB + (lane % CPR) * 16);
                *reinterpret_cast<f32x4*>(part + (wq * 32 + rr) * D + pass * (D / 2) + (lane % CPR) * 4) = v;
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the patch is rewritten by the next pass
        }
        return;
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const float inv = 1.f / l_tot[rb];
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i4 = 0; i4 < OC; ++i4) {
                bf16x4 o4;
#pragma unroll
                for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(oacc[db][rb][i4 * 4 + e] * inv);
                *reinterpret_cast<__attribute__((address_space(3))) bf16x4*>(patch + (rb * BR + lrow) * OROWB + (db * BR + i4 * 4 * KG + kg * 4) * 2) = o4;
            }
    }
    // lanes now read what other lanes of the same wave wrote: LDS operations of a wave complete in order
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __bf16* const outp = static_cast<__bf16*>(a.out);
#pragma unroll
    for (int p = 0; p < 32 / RPI; ++p) {
        const int rr = p * RPI + lane / CPR;
        const int row = wrow0 + rr;
        const u32x4 v = *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(patch + rr * OROWB + (lane % CPR) * 16);
        if (row < rows_total) {
            const int tok = div_g(row);
            const int head = g * G + (row - tok * G);
            *reinterpret_cast<u32x4*>(outp + ((long long)(s0 + tok) * Hq + head) * D + (lane % CPR) * 8) = v;
        }
    }
}

template <int D, int NG, int KG, bool SPLIT, class Work>
void launch_one(const AttnLaunch& a, const Work& wk, int entries, hipStream_t s) {
    const dim3 grid((unsigned)entries * a.kv_heads), block(256 * NG);
    hipLaunchKernelGGL((attn_bf16_kernel<D, NG, KG, SPLIT, Work>), grid, block, 0, s, a, wk);
}
template <class Work>
void launch_list(const AttnLaunch& a, const Work& wk, int entries, int variant, bool quarters, hipStream_t s) {
    const bool two = variant == kAttnVariantTwoGroups;
    if (a.head_dim == 64) {
        if (wk.splits > 1) launch_one<64, 1, 2, true>(a, wk, entries, s);
        else two ? launch_one<64, 2, 2, false>(a, wk, entries, s) : launch_one<64, 1, 2, false>(a, wk, entries, s);
    } else if (wk.splits > 1) {
        launch_one<128, 1, 2, true>(a, wk, entries, s);
    } else if (quarters) {
        two ? launch_one<128, 2, 4, false>(a, wk, entries, s) : launch_one<128, 1, 4, false>(a, wk, entries, s);
    } else {
        two ? launch_one<128, 2, 2, false>(a, wk, entries, s) : launch_one<128, 1, 2, false>(a, wk, entries, s);
    }
}

}  // namespace

hipError_t launch_attn_bf16(const AttnLaunch& a, const AttnWork& wk, int entries, int variant, bool quarters, hipStream_t s) {
    if (entries <= 0) return hipSuccess;
    wk.n_reqs <= kAttnReqStep ? launch_list(a, short_list(wk), entries, variant, quarters, s) : launch_list(a, wk, entries, variant, quarters, s);
    return hipGetLastError();
}

}  // namespace ragc
