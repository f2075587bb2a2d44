// bf16 prefix-cached paged attention for launches that cannot fill the chip with 128-row work
// items: decode steps, a few new tokens per request, one or two short requests, batches of
// half-empty items (plan_bf16 holds the rule).
//
// out[t,h,:] = softmax_j(scale * q[t,h,:].K_j) V_j over j = 0..prefix+i: cached keys from
// 16-token pool blocks through the block table (paper Sec. 5.1), the rest from the request's
// own fresh K/V (Sec. 3.2); the pass can also store that fresh K/V into its paged slots (Sec. 4).
//
// Mapping.  One workgroup = (request, kv head, 32 rows[, copy]); a row is a (new token, q head of
// the group) pair, token-major.  Its NW waves take every NW-th tile of 32 keys (two pool blocks)
// of the copy's key range, each with its own online softmax state, and the states are combined
// through LDS at the end.  A wave copies its tiles itself, straight into its own part of LDS
// (global_load_lds): K of the next tile during the P.V products of this one, V during its Q.K
// products.  There is no barrier in the loop, so a workgroup keeps 2 NW planes of 32 keys under
// way whatever its waves are doing -- which is what a launch this small is bound by.
//
// Products, layouts and softmax are those of attn_bf16_kernel: S^T = K.Q^T and O^T += V^T.P^T with
// v_mfma_f32_32x32x16_bf16, a lane owns one row and 16 of a tile's 32 keys.
#include "attn_bf16_common.h"
#include "attn_work.h"

namespace ragc {
namespace {

constexpr int TR = kAttnShortRows;  // rows per workgroup
constexpr int TK = 32;              // keys per tile

template <int D, int NW, bool SPLIT, class Work>
__global__ __launch_bounds__(64 * NW, 2) void attn_bf16_rows_kernel(AttnLaunch a, Work wk) {
    constexpr int CPR = D / 8;        // 16-byte chunks per K/V row
    constexpr int ROWB = D * 2;       // bytes per row
    constexpr int PLANEB = TK * ROWB; // one tile of K (or V)
    constexpr int RPI = 64 / CPR;     // rows one copy instruction covers
    constexpr int IPB = kBlock / RPI; // copy instructions per pool block and plane
    constexpr int NI = 2 * IPB;       // copy instructions per plane and tile
    constexpr int KSTEPS = D / 16;
    constexpr int DT = D / 32;
    constexpr int OCH = D / 4;        // 16-byte chunks of a fp32 output row
    constexpr int OWN = 8;            // up to so many rows of Q a wave brings for itself
    static_assert(TR * D * 4 == 2 * PLANEB, "a wave's output fills its tile buffers");
    __shared__ __attribute__((aligned(1024))) char smem[NW * 2 * PLANEB];
    __shared__ __attribute__((aligned(1024))) char qs[(NW * OWN > TR ? NW * OWN : TR) * ROWB];
    __shared__ float2 MLs[NW][TR];  // (max, sum) of every wave and row

    touch_args(a, wk);
    const int Hkv = a.kv_heads;
    int g, entry;
    split_block_id(a, blockIdx.x, &g, &entry);
    entry += wk.entry0;
    const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int S = SPLIT ? wk.splits : 1, sidx = SPLIT ? entry % S : 0;
    const WorkItem it = find_item(wk, SPLIT ? entry / S : entry, a.group, TR);
    const int G = a.group, N = it.new_len, P = it.prefix, s0 = it.new_start, Hq = a.q_heads;
    const uint32_t g_magic = a.group_magic;
    auto div_g = [&](int x) { return g_magic ? (int)__umulhi((uint32_t)x, g_magic) : x; };
    const int rows_total = N * G, row0 = it.tile * TR;

    const __bf16* __restrict__ q = static_cast<const __bf16*>(a.q);
    const __bf16* __restrict__ k_new = static_cast<const __bf16*>(a.k_new);
    const __bf16* __restrict__ v_new = static_cast<const __bf16*>(a.v_new);
    const __bf16* __restrict__ pool_k = static_cast<const __bf16*>(a.pool_k);
    const __bf16* __restrict__ pool_v = static_cast<const __bf16*>(a.pool_v);
    const int32_t* __restrict__ table = a.block_table + (long long)it.req * a.table_stride;

    const int rows_here = min(TR, rows_total - row0);
    const int kv_limit = P + div_g(row0 + rows_here - 1) + 1;  // keys [0, kv_limit) are visible to some row
    const int ntiles = (kv_limit + TK - 1) / TK;
    // copy sidx of S takes tiles [t_lo, t_hi); more copies than tiles: nothing for some, but each of them leaves a state
    const int t_lo = ntiles * sidx / S, t_hi = ntiles * (sidx + 1) / S;
    const int nsteps = t_hi - t_lo > w ? (t_hi - t_lo - w + NW - 1) / NW : 0;
    auto tile_of = [&](int step) { return t_lo + w + step * NW; };

    const int my_row = row0 + min(l32, rows_here - 1);  // rows past the end repeat the last one
    const int my_tok = div_g(my_row);
    const int my_vis = P + my_tok + 1;
    const int vis_min = P + div_g(row0) + 1;

    // block ids of this wave's tiles, 32 steps of two at a time, one per lane
    const int nblk = (kv_limit + kBlock - 1) / kBlock;
    auto id_at = [&](int step) { return table + min(tile_of(step + (lane >> 1)) * 2 + (lane & 1), nblk - 1); };
    int blk_base = 0, blk_vec;

    // Q: every wave needs all rows, copied to LDS behind its block ids and ahead of its first tile, 1 KiB per instruction.  Of
    // more than eight rows each wave brings a part for all: read by every wave from memory they were 64 KiB per workgroup, half
    // as much as the first tiles (one request of 1024 + 100 tokens 11.05 -> 10.6 us, 3000 + 64 of 2 heads, split, 12.9 ->
    // 11.6).  Up to eight, the rows of a decode step, are 16 KiB, and each wave brings its own: no wave waits for the others
    // (shared rows cost 4 of 4096 keys 0.9 us of 17.6), and Q does not wait for the first tiles (read into registers behind
    // them: 73 decode steps of 105 keys, 32/8 heads, 13.9 us against 12.65, 16 of 91-275 8.0 against 7.3, 4 of 4096, 64/8
    // heads, 19.3 against 19.0).
    const bool share_q = rows_here > OWN;
    {
        constexpr int QI = TR / RPI, NQ = QI > NW ? QI / NW : 1;  // with fewer pieces than waves some bring the same one
        constexpr int NQ_OWN = OWN / RPI;
        auto q_src = [&](int r) {
            const int row = row0 + min(r, rows_here - 1), tok = div_g(row);
            return q + ((long long)(s0 + tok) * Hq + g * G + (row - tok * G)) * D + ((lane % CPR) ^ swz<D>(r)) * 8;
        };
        const uint32_t q_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)qs;
        if (share_q) {
            const void* src[NQ];
#pragma unroll
            for (int x = 0; x < NQ; ++x) src[x] = q_src(RPI * ((w + x * NW) % QI) + lane / CPR);
            blk_vec = load_ahead_of_copies<NQ>(id_at(0), src, q_addr + w % QI * 1024, NW * 1024);
        } else {
            const void* src[NQ_OWN];
#pragma unroll
            for (int x = 0; x < NQ_OWN; ++x) src[x] = q_src(RPI * x + lane / CPR);
            blk_vec = load_ahead_of_copies<NQ_OWN>(id_at(0), src, q_addr + w * (OWN * ROWB), 1024);
        }
    }

    // ---- copies: lane i of an instruction brings row RPI c + i / CPR of a block, chunk (i % CPR) ^ swz(row)
    typedef __attribute__((address_space(3))) char lds_char;
    lds_char* const kbuf = (lds_char*)smem + w * (2 * PLANEB);
    lds_char* const vbuf = kbuf + PLANEB;
    const uint32_t k_addr = (uint32_t)(uintptr_t)kbuf;
    uint32_t pool_loff[IPB], new_loff[IPB];  // less what the instructions' own offsets add
#pragma unroll
    for (int c = 0; c < IPB; ++c) {
        const int row16 = RPI * c + lane / CPR;
        const int chunk = (lane % CPR) ^ swz<D>(row16);
        pool_loff[c] = (row16 * D + chunk * 8) * 2 - c * 1024;
        new_loff[c] = (row16 * Hkv * D + chunk * 8) * 2 - c * 1024;
    }
    auto copy_tile = [&](int step, bool is_k) {
        const __bf16* pool = is_k ? pool_k : pool_v;
        const __bf16* fresh = is_k ? k_new : v_new;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int kbase = tile_of(step) * TK + b * kBlock;
            const int blk = __builtin_amdgcn_readlane(blk_vec, 2 * (step - blk_base) + b);
            const uint32_t dst = k_addr + (is_k ? 0 : PLANEB) + b * kBlock * ROWB;
            if (kbase + kBlock <= P) {  // cached: one pool block
                dma_runs<IPB>(uniform_u64(pool + (long long)blk * a.block_stride + (long long)g * kBlock * D), pool_loff, dst);
            } else if (kbase >= P && kbase + kBlock <= kv_limit) {  // 16 fresh rows, all inside the horizon
                dma_runs<IPB>(uniform_u64(fresh + ((long long)(s0 + kbase - P) * Hkv + g) * D), new_loff, dst);
            } else {  // the prefix or the horizon ends inside, or before: keys past the horizon repeat the last visible one
#pragma unroll 1
                for (int c = 0; c < IPB; ++c) {
                    const int row16 = RPI * c + lane / CPR;
                    const int chunk = (lane % CPR) ^ swz<D>(row16);
                    const int key = min(kbase + row16, kv_limit - 1);
                    const __bf16* src = key < P ? pool + (long long)blk * a.block_stride + ((long long)g * kBlock + (key & (kBlock - 1))) * D
                                                : fresh + ((long long)(s0 + key - P) * Hkv + g) * D;
                    dma_16B_per_lane(src + chunk * 8, dst + RPI * c * ROWB);
                }
            }
        }
    };

    // ---- the first tile, as soon as its block ids are here
    if (nsteps > 0) {
        copy_tile(0, true);
        copy_tile(0, false);
        wait_vmcnt<2 * NI>();  // this wave's part of Q
    } else {
        wait_vmcnt<0>();
    }

    // ---- operand addresses (see attn_bf16_kernel)
    int koff[KSTEPS], voff[2][DT];
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) koff[ks] = l32 * ROWB + (((2 * ks + hf) ^ swz<D>(l32)) << 4);
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const int row = 8 * h2 + 4 * hf + ((lane & 15) >> 2);
            const int elem = dt * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
            voff[h2][dt] = row * ROWB + ((((elem >> 3)) ^ swz<D>(row)) << 4) + (elem & 7) * 2;
        }

    if (share_q) block_barrier();  // every wave's part of Q has landed
    lds_char* const qbuf = (lds_char*)qs + (share_q ? 0 : w * (OWN * ROWB));
    const int q_row = share_q ? l32 : min(l32, OWN - 1);
    bf16x8 qreg[KSTEPS];
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks)
        qreg[ks] = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(qbuf + q_row * ROWB + (((2 * ks + hf) ^ swz<D>(q_row)) << 4));

    f32x16 oacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[dt][i] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;  // reference exponent, at most 2^8 below the maximum so far; l is this lane's part
    const float c = a.scale_log2e;

    auto do_tile = [&](int step, auto more_c) {
        constexpr bool MORE = decltype(more_c)::value;  // another tile follows
        wait_vmcnt<NI>();  // K is here, V may be under way
        f32x16 s;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            const bf16x8 kk = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(kbuf + koff[ks]);
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk, qreg[ks], s, 0, 0, 0);
        }
        if (MORE) {
            if (step + 1 - blk_base >= 32) {
                blk_base = step + 1;
                blk_vec = *id_at(step + 1);
                asm volatile("" ::"v"(blk_vec));  // the wait for this load stays inside the branch
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this tile's K has been read
            copy_tile(step + 1, true);
        }
        const int base = tile_of(step) * TK;
        if (base + TK > vis_min) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (base + (i >> 2) * 8 + hf * 4 + (i & 3) >= my_vis) s[i] = -INFINITY;
        }
        float mx = s[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
        if (__builtin_amdgcn_ballot_w64(mx * c > m_run + kRescaleThreshold) != 0) {
            mx = fmaxf(mx, other_half(mx)) * c;
            const bool raise = mx > m_run + kRescaleThreshold;  // true on a row's first visible tile (m_run = -inf)
            const float alpha = raise ? __builtin_amdgcn_exp2f(m_run - mx) : 1.f;
            m_run = raise ? mx : m_run;
            l_run *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[dt][i] *= alpha;
        }
        const float m_sub = m_run == -INFINITY ? 0.f : m_run;  // a row without a visible key yet: exp2(-inf - 0) = 0
        float psum = 0.f;  // over the bf16-rounded probabilities, the weights of the P.V product
        bf16x8 pb[2];
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            const float p0 = __builtin_amdgcn_exp2f(s[i] * c - m_sub);
            const float p1 = __builtin_amdgcn_exp2f(s[i + 1] * c - m_sub);
            const bf16x2 pp = {(__bf16)p0, (__bf16)p1};
            psum = __builtin_amdgcn_fdot2_f32_bf16(pp, kOnes2, psum, false);
            pb[i >> 3][i & 7] = pp[0];
            pb[i >> 3][(i & 7) + 1] = pp[1];
        }
        l_run += psum;
        wait_vmcnt<MORE ? NI : 0>();  // V is here, the next K may be under way
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                lds_char* const vb = vbuf + kk * 16 * ROWB;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(vb + voff[0][dt]));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(vb + voff[1][dt]));
                const bf16x8 va = __builtin_shufflevector(__builtin_bit_cast(bf16x4, lo), __builtin_bit_cast(bf16x4, hi), 0, 1, 2, 3, 4, 5, 6, 7);
                oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[kk], oacc[dt], 0, 0, 0);
            }
        if (MORE) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this tile's V has been read
            copy_tile(step + 1, false);
        }
    };
    if (nsteps > 0) {
        for (int step = 0; step + 1 < nsteps; ++step) do_tile(step, std::true_type{});
        do_tile(nsteps - 1, std::false_type{});
    }

    // ---- fused append: this workgroup owns the tokens whose first row (head 0 of the group) it holds
    if (a.fused_append && sidx == S - 1) {
        const int tok_lo = div_g(row0 + G - 1), tok_hi = min(N - 1, div_g(row0 + TR - 1));
        __bf16* wkp = static_cast<__bf16*>(a.pool_k);
        __bf16* wvp = static_cast<__bf16*>(a.pool_v);
        for (int idx = tid; idx < (tok_hi - tok_lo + 1) * CPR; idx += 64 * NW) {
            const int tok = tok_lo + idx / CPR, ch = idx % CPR, pos = P + tok;
            const long long from = ((long long)(s0 + tok) * Hkv + g) * D + ch * 8;
            const u32x4 kk = *reinterpret_cast<const u32x4*>(k_new + from), vv = *reinterpret_cast<const u32x4*>(v_new + from);
            const long long to = (long long)table[pos >> 4] * a.block_stride + ((long long)g * kBlock + (pos & 15)) * D + ch * 8;
            *reinterpret_cast<u32x4*>(wkp + to) = kk;
            *reinterpret_cast<u32x4*>(wvp + to) = vv;
        }
    }

    // ---- combine the waves' states: O = sum_w O_w 2^(m_w - m), l = sum_w l_w 2^(m_w - m), m = max_w m_w.  Every wave
    // leaves its O in its own part of LDS, [row][chunk of 4 columns], chunks XORed with the row against bank conflicts.
    // l is exactly 0 in a wave that has seen no key of the row, and its O counts as 0; m = -inf does not say so: a
    // wave whose scores were all NaN still has it, next to l = NaN and O = NaN, which must reach the output.
    // All waves' pieces are read without a look at their weights: a branch per wave made a trip to LDS of each.
    l_run += other_half(l_run);
    if (hf == 0) MLs[w][l32] = float2{m_run, l_run};
    if (l_run == 0.f) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 16; ++i) oacc[dt][i] = 0.f;
    }
    if (l32 < rows_here) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const f32x4 v = {oacc[dt][i4 * 4], oacc[dt][i4 * 4 + 1], oacc[dt][i4 * 4 + 2], oacc[dt][i4 * 4 + 3]};
                *reinterpret_cast<__attribute__((address_space(3))) f32x4*>(kbuf + l32 * (D * 4) + (((dt * 8 + i4 * 2 + hf) ^ (l32 & (OCH - 1))) << 4)) = v;
            }
    }
    __syncthreads();
    constexpr int TPR = CPR;  // threads per row: 8 columns each
    for (int idx = tid; idx < rows_here * TPR; idx += 64 * NW) {
        const int r = idx / TPR, c8 = idx % TPR;
        float2 ml[NW];
        float m = -INFINITY, l = 0.f;
#pragma unroll
        for (int x = 0; x < NW; ++x) {
            ml[x] = MLs[x][r];
            m = fmaxf(m, ml[x].x);
        }
        f32x4 o[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int x = 0; x < NW; ++x) {
            // a wave, or every one of a copy, may have seen no key of the row
            const float wgt = ml[x].y == 0.f ? 0.f : __builtin_amdgcn_exp2f(ml[x].x - m);
            l += ml[x].y * wgt;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4 v = *reinterpret_cast<const __attribute__((address_space(3))) f32x4*>(
                    (lds_char*)smem + x * (2 * PLANEB) + r * (D * 4) + (((2 * c8 + h) ^ (r & (OCH - 1))) << 4));
#pragma unroll
                for (int e = 0; e < 4; ++e) o[h][e] += v[e] * wgt;
            }
        }
        if (SPLIT) {
            float* const part = static_cast<float*>(a.partial) + ((long long)(wk.part_base + entry) * Hkv + g) * (TR * (D + 2));
            if (c8 == 0) *reinterpret_cast<float2*>(part + TR * D + r * 2) = float2{m, l};
            *reinterpret_cast<f32x4*>(part + r * D + c8 * 8) = o[0];
            *reinterpret_cast<f32x4*>(part + r * D + c8 * 8 + 4) = o[1];
        } else {
            const float inv = 1.f / l;
            const int row = row0 + r, tok = div_g(row);
            bf16x8 ob;
#pragma unroll
            for (int e = 0; e < 8; ++e) ob[e] = (__bf16)(o[e >> 2][e & 3] * inv);
            *reinterpret_cast<bf16x8*>(static_cast<__bf16*>(a.out) + ((long long)(s0 + tok) * Hq + g * G + (row - tok * G)) * D + c8 * 8) = ob;
        }
    }
}

// Combines the S partial results of every row of a split work item of ROWS rows, of either kernel (see the end of
// attn_bf16_rows_kernel for the layout): out = sum_s O_s 2^(m_s - m) / sum_s l_s 2^(m_s - m), m = max_s m_s.
// One workgroup per (item, kv head, run of 256 / (D/4) rows): 4 consecutive d of one row per thread.
template <int D, int ROWS, class Work>
__global__ __launch_bounds__(256) void attn_bf16_merge_kernel(AttnLaunch a, Work wk) {
    constexpr int TPR = D / 4;          // threads per row
    constexpr int RPW = 256 / TPR;      // rows per workgroup
    constexpr int CHUNKS = ROWS / RPW;    // workgroups per (entry, kv head)
    const int Hkv = a.kv_heads;
    const int chunk = blockIdx.x % CHUNKS;
    const int g = (blockIdx.x / CHUNKS) % Hkv;
    const int lead = blockIdx.x / (CHUNKS * Hkv) + wk.entry0 / wk.splits;
    const WorkItem it = find_item(wk, lead, a.group, ROWS);
    const int S = wk.splits;
    const int G = a.group;
    const uint32_t g_magic = a.group_magic;
    auto div_g = [&](int x) { return g_magic ? (int)__umulhi((uint32_t)x, g_magic) : x; };
    const int rows_total = it.new_len * G;
    const int row0 = it.tile * ROWS;
    const int rows_here = min(ROWS, rows_total - row0);
    constexpr int PART = ROWS * (D + 2);
    const float* const part0 = static_cast<const float*>(a.partial) + ((long long)(wk.part_base + lead * S) * Hkv + g) * PART;
    const long long copy_stride = (long long)Hkv * PART;
    const int d4 = threadIdx.x % TPR;
    __bf16* const outp = static_cast<__bf16*>(a.out);
    const int r = chunk * RPW + threadIdx.x / TPR;
    if (r < rows_here) {
        // one round trip: every copy's (max, sum) and O piece are requested before any is used
        float mc[kAttnMaxSplits], lc[kAttnMaxSplits];
        f32x4 oc[kAttnMaxSplits];
#pragma unroll
        for (int c = 0; c < kAttnMaxSplits; ++c) {
            mc[c] = -INFINITY;  // a copy that does not exist weighs 0
            lc[c] = 0.f;
            oc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (c < S) {
                const float* pc = part0 + c * copy_stride;
                const float2 ml = *reinterpret_cast<const float2*>(pc + ROWS * D + r * 2);
                mc[c] = ml.x;
                lc[c] = ml.y;
                oc[c] = *reinterpret_cast<const f32x4*>(pc + r * D + d4 * 4);
            }
        }
        float m = -INFINITY;
#pragma unroll
        for (int c = 0; c < kAttnMaxSplits; ++c) m = fmaxf(m, mc[c]);
        float l = 0.f;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < kAttnMaxSplits; ++c) {
            const float wgt = mc[c] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mc[c] - m);  // a copy may hold no visible key of the row
            l += lc[c] * wgt;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += oc[c][e] * wgt;
        }
        const float inv = 1.f / l;
        const int row = row0 + r;
        const int tok = div_g(row);
        const int head = g * G + (row - tok * G);
        bf16x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(acc[e] * inv);
        *reinterpret_cast<bf16x4*>(outp + ((long long)(it.new_start + tok) * a.q_heads + head) * D + d4 * 4) = o4;
    }
}

template <int D, int NW, bool SPLIT, class Work>
void launch_one(const AttnLaunch& a, const Work& wk, int entries, hipStream_t s) {
    const dim3 grid((unsigned)entries * a.kv_heads), block(64 * NW);
    hipLaunchKernelGGL((attn_bf16_rows_kernel<D, NW, SPLIT, Work>), grid, block, 0, s, a, wk);
}
template <class Work>
void launch_list(const AttnLaunch& a, const Work& wk, int entries, int waves, hipStream_t s) {
    const bool d64 = a.head_dim == 64;
    if (wk.splits > 1) d64 ? launch_one<64, 8, true>(a, wk, entries, s) : launch_one<128, 8, true>(a, wk, entries, s);
    else if (waves == 4) d64 ? launch_one<64, 4, false>(a, wk, entries, s) : launch_one<128, 4, false>(a, wk, entries, s);
    else d64 ? launch_one<64, 8, false>(a, wk, entries, s) : launch_one<128, 8, false>(a, wk, entries, s);
}

template <int D, int ROWS, class Work>
void launch_merge_one(const AttnLaunch& a, const Work& wk, int entries, hipStream_t s) {
    const dim3 grid((unsigned)(entries / wk.splits) * a.kv_heads * (ROWS * D / 1024));
    hipLaunchKernelGGL((attn_bf16_merge_kernel<D, ROWS, Work>), grid, dim3(256), 0, s, a, wk);
}
template <class Work>
void launch_merge(const AttnLaunch& a, const Work& wk, int entries, int rows, hipStream_t s) {
    const bool d64 = a.head_dim == 64;
    if (rows == TR) d64 ? launch_merge_one<64, TR>(a, wk, entries, s) : launch_merge_one<128, TR>(a, wk, entries, s);
    else d64 ? launch_merge_one<64, kAttnRowsPerItem>(a, wk, entries, s) : launch_merge_one<128, kAttnRowsPerItem>(a, wk, entries, s);
}

}  // namespace

hipError_t launch_attn_bf16_rows(const AttnLaunch& a, const AttnWork& wk, int entries, int waves, hipStream_t s) {
    if (entries <= 0) return hipSuccess;
    wk.n_reqs <= kAttnReqStep ? launch_list(a, short_list(wk), entries, waves, s) : launch_list(a, wk, entries, waves, s);
    return hipGetLastError();
}

hipError_t launch_attn_bf16_merge(const AttnLaunch& a, const AttnWork& wk, int entries, int rows, hipStream_t s) {
    if (entries <= 0) return hipSuccess;
    wk.n_reqs <= kAttnReqStep ? launch_merge(a, short_list(wk), entries, rows, s) : launch_merge(a, wk, entries, rows, s);
    return hipGetLastError();
}

}  // namespace ragc
