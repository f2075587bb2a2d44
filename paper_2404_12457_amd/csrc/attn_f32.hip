// fp32 prefix-cached paged prefill attention on the matrix cores of gfx950.
//
// out[t,h,:] = softmax_j(scale * q[t,h,:].K_j) V_j over j = 0..prefix+i, where the
// first `prefix` keys are gathered from 16-token pool blocks through the request's
// block table (paper Sec. 5.1: non-contiguous blocks referenced by tree nodes) and
// the rest are the request's own fresh K/V (Sec. 3.2: only the request tokens are
// computed).  Inputs, softmax and sums are fp32; products are fp32 (16 rows), or of three-part
// bf16 splits of both operands, six of the nine products of parts summed in fp32 (32 rows).
//
// Two kernels (the rule between them is plan_f32).  One workgroup = (request, kv head, 16 or 32 rows);
// a row is a (new token, q head of the group) pair, token-major, so the heads of a GQA group share
// every K/V read.  Its NW waves take every NW-th tile of 16 keys -- one pool block -- with an online
// softmax state of their own each, and the states are combined through LDS at the end: no barrier
// and no shared tile in the key loop.  Each wave copies its own tile straight into its own part of
// LDS (global_load_lds), K during the P.V products of the tile before, V during the Q.K products.
//
// attn_f32_kernel, 16 rows: fp32 matrix cores (plain_rows), 64 flop per cycle and SIMD (157 TFLOP/s
// on the chip).  A 16-key tile at head_dim 128 is 64 products, 2048 cycles, and the loop runs at 0.8
// of that with two waves per SIMD; the rest of a small call is the 5 us before the first tile and
// after the last.  So Q, which each wave would wait for by itself, comes through LDS once per
// workgroup, behind the block ids and ahead of the first tile's copies: one request of 256 + 32
// tokens, 4 heads of 64: 7.8 -> 7.15 us (27 with plain FMAs from shared tiles); 7 of 2-4 new tokens,
// 16 heads of 64: 7.9 -> 6.65.  Tried: K read from global memory in operand order instead of through LDS costs a
// cache access per lane (41 on average per load instruction, 2600 cycles per tile and CU); K staged
// through registers and three waves per SIMD: both 5-10 % slower.
//
// attn_f32_split_kernel, 32 rows: bf16 matrix cores, without rounding an operand.  A float is the
// exact sum of three bf16 numbers, x = x0 + x1 + x2 (8 bits of the significand each), and of the nine
// products of two such sums the six above 2^-24 of the whole are taken, x0y0, x0y1, x1y0, x1y1,
// x0y2, x2y0, each exact in fp32, where they are summed.  The three left out are together below
// 2^-24 of |x||y|, less than the rounding of one fp32 product.  Against 64 bits, 24 batches: relative
// error 2.65e-7 to 4.66e-7 where the fp32 products have 2.90e-7 to 5.50e-7, lower on each.
// What bounds it: a tile and 32 rows at head_dim 128 are 1536 cycles of products (4096 with fp32
// products) and about 400 vector instructions, most of them the split of K and V, and a SIMD's two
// waves overlap little of one with the other (a probe of products with four vector instructions
// behind each: the sum of both times but a tenth; with the split of one step placed between the
// products of the step before, 2 % slower than in the compiler's order).  4 requests of 512-1024
// cached and 32-100 new tokens, 32/8 heads: 36.1 -> 28.0 us.
#include "attn_bf16_common.h"
#include "attn_work.h"

namespace ragc {
namespace {

constexpr int KT = kBlock;     // keys per tile
constexpr float kRaise = 8.f;  // log2 units a row's reference exponent may lag behind its maximum
constexpr float kTiny = 0x1p-100f;  // of operands below 2^-110, parts are below the smallest bf16 number
constexpr float kLift = 0x1p24f;    // of the probabilities, which are normal down to 2^-126: all three parts are then above it

typedef __attribute__((ext_vector_type(2))) float f32x2;
constexpr int kA[6] = {2, 0, 1, 1, 0, 0}, kB[6] = {0, 2, 1, 0, 1, 0};  // the parts of the six products, smallest first

// 16 rows of a work item with fp32 products (v_mfma_f32_16x16x4_f32): row tile `tile` of 16 rows.
//   S^T[key][row] = K . Q^T    A: lane (key l16, group kg) holds K[key][16 j + 4 kg + e], a
//                              16-byte read per j; B: Q with the same order of the contraction
//   O^T[d][row]  += V^T . P^T  A: lane (l16, kg) holds V[4 kg + i][64 c + 4 l16 + e], a 16-byte
//                              read per (c, i) serves four products (e); B: P^T, which is the
//                              accumulator of S^T as it stands (lane: row l16, keys 4 kg + i)
template <int D, int NW>
__device__ __forceinline__ void plain_rows(const AttnLaunch& a, const WorkItem& it, int g, int tile, bool append, char* smem,
                                           char* qs, float (*Ms)[16], float (*Ls)[16]) {
    constexpr int TR = 16;                 // rows
    constexpr int KJ = D / 16;             // 16-byte reads of a K row per lane
    constexpr int VC = D / 64;             // 16-byte reads of a V row per lane
    constexpr int CPR = D / 4;             // 16-byte chunks per row
    constexpr int ROWB = D * 4;            // bytes per row
    constexpr int PLANEB = KT * ROWB;      // one tile of K (or V)
    constexpr int RPI = 64 / CPR;          // rows one copy instruction covers
    constexpr int NI = KT / RPI;           // copy instructions per plane and tile
    constexpr int OSTRIDE = D + 4;         // floats per output row in LDS
    static_assert(TR * OSTRIDE * 4 <= 2 * PLANEB, "a wave's output fits its tile buffers");
    const int Hkv = a.kv_heads;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int P = it.prefix, N = it.new_len, s0 = it.new_start, G = a.group;
    const uint32_t g_magic = a.group_magic;
    auto div_g = [&](uint32_t x) { return g_magic ? (int)__umulhi(x, g_magic) : (int)x; };  // exact while x * G < 2^32
    const long long row0 = (long long)tile * TR;
    const int rows_here = (int)min((long long)TR, (long long)N * G - row0);
    const int tok0 = row0 * G >> 32 ? (int)(row0 / G) : div_g((uint32_t)row0);  // row 0 of the tile: token tok0,
    const int h0 = (int)(row0 - (long long)tok0 * G);                          // head h0 of the group

    const float* __restrict__ q = static_cast<const float*>(a.q);
    const float* __restrict__ k_new = static_cast<const float*>(a.k_new);
    const float* __restrict__ v_new = static_cast<const float*>(a.v_new);
    const float* __restrict__ pool_k = static_cast<const float*>(a.pool_k);
    const float* __restrict__ pool_v = static_cast<const float*>(a.pool_v);
    const int32_t* __restrict__ table = a.block_table + (long long)it.req * a.table_stride;

    const int l16 = lane & 15, kg = lane >> 4;
    const int kv_limit = P + tok0 + div_g(h0 + rows_here - 1) + 1;  // keys [0, kv_limit) are visible to some row
    const int ntiles = (kv_limit + KT - 1) / KT;
    const int nsteps = ntiles > w ? (ntiles - w + NW - 1) / NW : 0;  // this wave takes tiles w, w + NW, ...
    const int my_vis = P + tok0 + div_g(h0 + min(l16, rows_here - 1)) + 1;  // rows past the end repeat the last one and are not stored
    const int vis_min = P + tok0 + 1;  // tiles below need no mask

    // block ids of this wave's tiles, 64 steps at a time, one per lane; and Q, which every wave needs, copied to LDS once and
    // shared (swizzled as K is): the first copies wait for neither.  Up to four rows are less than the wait for the other waves
    // and come straight to the registers (24 requests of 16-26 + 1-2 tokens, 32 heads of 128: 13.3 us shared, 12.85 so).
    int blk_base = 0, blk_vec;
    const bool share_q = rows_here > 4;
    f32x4 qreg[KJ];
    if (share_q) {
        constexpr int QI = TR / RPI, NQ = QI > NW ? QI / NW : 1;  // with fewer pieces than waves some bring the same one
        const void* src[NQ];
#pragma unroll
        for (int x = 0; x < NQ; ++x) {
            const int r = RPI * ((w + x * NW) % QI) + lane / CPR, row = h0 + min(r, rows_here - 1), tok = div_g(row);
            src[x] = q + ((long long)(s0 + tok0 + tok) * a.q_heads + g * G + (row - tok * G)) * D + ((lane % CPR) ^ r) * 4;
        }
        blk_vec = load_ahead_of_copies<NQ>(table + min(w + lane * NW, ntiles - 1), src,
                                           (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)qs + w % QI * 1024, NW * 1024);
    } else {
        blk_vec = table[min(w + lane * NW, ntiles - 1)];
        const int tok = div_g(h0 + min(l16, rows_here - 1));
        const float* qp = q + ((long long)(s0 + tok0 + tok) * a.q_heads + g * G + (h0 + min(l16, rows_here - 1) - tok * G)) * D + kg * 4;
#pragma unroll
        for (int j = 0; j < KJ; ++j) qreg[j] = *reinterpret_cast<const f32x4*>(qp + j * 16);
        asm volatile("" ::"v"(blk_vec));
#pragma unroll
        for (int j = 0; j < KJ; ++j) asm volatile("" ::"v"(qreg[j]));
        wait_vmcnt<0>();
    }

    // Copies: lane i of instruction n brings row RPI n + i / CPR of the tile.  K rows are stored with their chunk
    // index XORed with the row (on the global side), so that the 16 keys of an operand read hit different banks.
    typedef __attribute__((address_space(3))) char lds_char;
    typedef const __attribute__((address_space(3))) f32x4 lds_f32x4;
    lds_char* const kbuf = (lds_char*)smem + w * (2 * PLANEB);
    lds_char* const vbuf = kbuf + PLANEB;
    const uint32_t k_addr = (uint32_t)(uintptr_t)kbuf, v_addr = k_addr + PLANEB;
    const int new_row = Hkv * D;                                    // elements between fresh rows
    const long long new_off = ((long long)(s0 - P) * Hkv + g) * D;  // of the fresh row at position 0
    auto copy_tile = [&](int step, bool is_k) {
        const int base = (w + step * NW) * KT;
        const long long boff = (long long)__builtin_amdgcn_readlane(blk_vec, step - blk_base) * a.block_stride + (long long)g * kBlock * D;
        const float* pool = is_k ? pool_k : pool_v;
        const float* fresh = is_k ? k_new : v_new;
        const uint32_t dst = is_k ? k_addr : v_addr;
        auto copy_runs = [&](uint64_t src, int row_bytes) {  // four instructions, 4 KiB of LDS, at a time
#pragma unroll
            for (int n0 = 0; n0 < NI; n0 += 4) {
                uint32_t off[4];
#pragma unroll
                for (int n = 0; n < 4; ++n) {
                    const int row = RPI * (n0 + n) + lane / CPR, chunk = lane % CPR;
                    off[n] = (uint32_t)(row * row_bytes + (is_k ? chunk ^ row : chunk) * 16 - n * 1024);
                }
                dma_runs<4>(src, off, dst + n0 * 1024);
            }
        };
        if (base + KT <= P) {  // one pool block: uniform base, per-lane constant offset
            copy_runs(uniform_u64(pool + boff), ROWB);
        } else if (base >= P && base + KT <= kv_limit) {  // fresh rows, all inside the horizon
            copy_runs(uniform_u64(fresh + new_off + (long long)base * new_row), new_row * 4);
        } else {  // the prefix or the horizon ends inside: source per row; keys past the horizon repeat the last visible one
#pragma unroll 1
            for (int n = 0; n < NI; ++n) {
                const int row = RPI * n + lane / CPR, chunk = is_k ? (lane % CPR) ^ row : lane % CPR;
                const int key = base + row;
                const float* src = key < P ? pool + boff + row * D : fresh + new_off + (long long)min(key, kv_limit - 1) * new_row;
                dma_16B_per_lane(src + chunk * 4, dst + n * 1024);
            }
        }
    };
    if (nsteps > 0) {
        copy_tile(0, true);
        wait_vmcnt<NI>();  // this wave's part of Q
    } else {
        wait_vmcnt<0>();
    }
    int koff[KJ];  // this lane's K reads
#pragma unroll
    for (int j = 0; j < KJ; ++j) koff[j] = l16 * ROWB + (((4 * j + kg) ^ l16) << 4);
    const int voff = kg * 4 * ROWB + l16 * 16;

    if (share_q) {
        block_barrier();  // every wave's part of Q has landed
#pragma unroll
        for (int j = 0; j < KJ; ++j) qreg[j] = *reinterpret_cast<lds_f32x4*>((lds_char*)qs + koff[j]);
    }

    // V of the first tile behind the barrier: a wave whose tile takes a source per row issues its copies for half a microsecond,
    // and all waves would wait for it (23 requests of 53-161 + 5 tokens, 4 heads of 128: 10.4 us, so 9.7; 23 of 26-105 + 2, 64/8
    // heads, 9.0 and 8.1).
    if (nsteps > 0) copy_tile(0, false);

    f32x4 oacc[VC][4];
#pragma unroll
    for (int c = 0; c < VC; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) oacc[c][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;  // l: this lane's keys only
    const float sc = a.scale_log2e;

    auto do_tile = [&](int step, auto more_c) {
        constexpr bool MORE = decltype(more_c)::value;  // another tile follows
        wait_vmcnt<NI>();  // K is here, V may be under way
        // Two chains of products side by side (a product waits for the one before it), and two after one another (each rounds
        // at the size of its sum so far).  Against 64 bits, 4 requests of 512-1024 + 32-100 tokens, five draws: relative error
        // 4.5e-7 to 4.7e-7, largest 4.2e-6 to 6.3e-6; with one pair 5.8e-7 to 6.1e-7 and 6.0e-6 to 1.6e-5, in the same time.
        // More side by side cost time where two waves share a SIMD (eight: 2 % on 43 batches, up to 24 %).
        constexpr int CH = 4;
        f32x4 sp[CH];
#pragma unroll
        for (int x = 0; x < CH; ++x) sp[x] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < KJ; ++j) {
            const f32x4 kr = *reinterpret_cast<lds_f32x4*>(kbuf + koff[j]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                f32x4& x = sp[2 * (j / (KJ / 2)) + e % 2];
                x = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[e], qreg[j][e], x, 0, 0, 0);
            }
        }
#pragma unroll
        for (int n = CH / 2; n > 0; n /= 2)
#pragma unroll
            for (int x = 0; x < n; ++x) sp[x] += sp[x + n];
        if (MORE) {
            if (step + 1 - blk_base >= 64) {
                blk_base = step + 1;
                blk_vec = table[min(w + (step + 1 + lane) * NW, ntiles - 1)];
                asm volatile("" ::"v"(blk_vec));  // the wait for this load stays inside the branch
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this tile's K has been read
            copy_tile(step + 1, true);
        }
        f32x4 s;
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] = sp[0][i] * sc;
        const int base = (w + step * NW) * KT;
        if (base + KT > vis_min) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (base + kg * 4 + i >= my_vis) s[i] = -INFINITY;
        }
        // the reference exponent of a row is raised only when a score exceeds it by more than 2^8 (or on the
        // row's first visible key); the four lanes of a row keep the same one
        float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
        if (__builtin_amdgcn_ballot_w64(mx > m_run + kRaise) != 0) {
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const bool raise = mx > m_run + kRaise;
            const float alpha = raise ? __builtin_amdgcn_exp2f(m_run - mx) : 1.f;  // first visible key: exp2(-inf) = 0
            m_run = raise ? mx : m_run;
            l_run *= alpha;
#pragma unroll
            for (int c = 0; c < VC; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < 4; ++i) oacc[c][e][i] *= alpha;
        }
        const float m_sub = m_run == -INFINITY ? 0.f : m_run;  // a row without a visible key yet: exp2(-inf - 0) = 0
        wait_vmcnt<MORE ? NI : 0>();  // V is here, the next K may be under way
        float p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(s[i] - m_sub);
        l_run += (p[0] + p[1]) + (p[2] + p[3]);
        if (!MORE && base + KT > kv_limit) {
            // rows past the horizon hold the last visible V again, which 0 times its probability only takes out while
            // it is finite (the K rows are masked whatever they hold)
            for (int x = lane; x < (base + KT - kv_limit) * CPR; x += 64)
                *reinterpret_cast<__attribute__((address_space(3))) f32x4*>(vbuf + (kv_limit - base) * ROWB + x * 16) = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < VC; ++c) {
                const f32x4 vr = *reinterpret_cast<lds_f32x4*>(vbuf + voff + i * ROWB + c * 256);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    oacc[c][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[e], p[i], oacc[c][e], 0, 0, 0);
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this tile's V has been read
        if (MORE) copy_tile(step + 1, false);
    };
    if (nsteps > 0) {
        for (int step = 0; step + 1 < nsteps; ++step) do_tile(step, std::true_type{});
        do_tile(nsteps - 1, std::false_type{});
    }

    // fused append: this workgroup owns the tokens whose first row (head 0 of the group) it holds
    if (append && a.fused_append) {
        const int tok_lo = tok0 + (h0 != 0), tok_hi = min(N - 1, tok0 + div_g(h0 + TR - 1));
        float* wk_pool = static_cast<float*>(a.pool_k);
        float* wv_pool = static_cast<float*>(a.pool_v);
        for (int idx = tid; idx < (tok_hi - tok_lo + 1) * (D / 4); idx += 64 * NW) {
            const int tok = tok_lo + idx / (D / 4), c4 = idx % (D / 4);
            const int pos = P + tok;
            const long long src = ((long long)(s0 + tok) * Hkv + g) * D + c4 * 4;
            const long long dst = (long long)table[pos >> 4] * a.block_stride + ((long long)g * kBlock + (pos & 15)) * D + c4 * 4;
            *reinterpret_cast<f32x4*>(wk_pool + dst) = *reinterpret_cast<const f32x4*>(k_new + src);
            *reinterpret_cast<f32x4*>(wv_pool + dst) = *reinterpret_cast<const f32x4*>(v_new + src);
        }
    }

    // combine the waves' states (each left in the wave's own part of LDS): out = sum_w O_w 2^(m_w - m) / sum_w l_w 2^(m_w - m)
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    float* const Os = reinterpret_cast<float*>(smem);
    constexpr int OWAVE = 2 * PLANEB / 4;
    if (kg == 0) {
        Ms[w][l16] = m_run;
        Ls[w][l16] = l_run;
    }
#pragma unroll
    for (int c = 0; c < VC; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<f32x4*>(Os + (w * OWAVE + l16 * OSTRIDE + 64 * c + 16 * kg + 4 * i)) =
                f32x4{oacc[c][0][i], oacc[c][1][i], oacc[c][2][i], oacc[c][3][i]};
    __syncthreads();
    float* __restrict__ out = static_cast<float*>(a.out);
    for (int idx = tid; idx < TR * (D / 4); idx += 64 * NW) {
        const int r = idx / (D / 4), c4 = idx % (D / 4);
        if (r >= rows_here) break;
        float m = -INFINITY;
#pragma unroll
        for (int x = 0; x < NW; ++x) m = fmaxf(m, Ms[x][r]);
        float l = 0.f;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int x = 0; x < NW; ++x) {
            const float wgt = Ms[x][r] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(Ms[x][r] - m);  // a wave may have seen no key of the row
            l += Ls[x][r] * wgt;
            const f32x4 ox = *reinterpret_cast<const f32x4*>(Os + (x * OWAVE + r * OSTRIDE + c4 * 4));
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] += ox[e] * wgt;
        }
        const float inv = 1.f / l;
        const int dtok = div_g(h0 + r), head = g * G + h0 + r - dtok * G;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] *= inv;
        *reinterpret_cast<f32x4*>(out + ((long long)(s0 + tok0 + dtok) * a.q_heads + head) * D + c4 * 4) = o;
    }
}

template <int D, int NW, class Work>
__global__ __launch_bounds__(64 * NW, 2) void attn_f32_kernel(AttnLaunch a, Work wk) {
    __shared__ __attribute__((aligned(1024))) char smem[NW * 2 * KT * D * 4], qs[16 * D * 4];
    __shared__ float Ms[NW][16], Ls[NW][16];
    touch_args(a, wk);
    int g, entry;
    split_block_id(a, blockIdx.x, &g, &entry);
    entry += wk.entry0;
    const WorkItem it = find_item(wk, entry, a.group, 16);
    plain_rows<D, NW>(a, it, g, it.tile, true, smem, qs, Ms, Ls);
}

// ---- the split products
//   S^T[key][row] = K . Q^T    v_mfma_f32_16x16x32_bf16, two halves of 16 rows; A: lane (key
//                              l16, group kg) holds K[key][32 j + {4 kg + e, 16 + 4 kg + e}];
//                              B: Q with the same order of the contraction
//   O^T[d][row]  += V^T . P^T  v_mfma_f32_32x32x16_bf16; B: P^T after one v_permlane16_swap per
//                              score register (lane: row l32, keys 8 hf + j); A: lane (l32, hf)
//                              holds V[8 hf + j][64 u + 2 l32 + t] for accumulator 2 u + t
// and a lane ends up with pairs of output columns of its row.
//
// What no split into bf16 numbers keeps is computed again by the workgroup, all its rows with fp32 products, as if it had never
// split.  Products, sums and conversions keep denormals here (the exponential alone does not), so a part is lost only below the
// smallest bf16 number, 2^-133: at most 2^-134 of an operand, and nothing above 2^-110.  It shows
//   - by an output that is not finite: infinities and NaN, or K or V that round to infinity;
//   - by an output below 2^-100: V as small, whose 2^-134 count there;
//   - by Q: 2^-134 of K count in a score only where Q (times softmax_scale) is above 2^96, and Q itself loses below 2^-110.
// Probabilities go down to 2^-126 next to any V, so they are lifted by 2^24 before their split, and their sums with them.  What
// does not show is a V below 2^-134, of which nothing is left: it counts as 0.  An output of 0 says nothing, as it is what the
// columns that pad a head give; to look through V for it doubled the time of such heads.
// The looks at Q and at the outputs take 0.1 us of a workgroup, the lift half a percent of a long range: 30 requests of 16-34 + 35-71
// tokens, 28/4 heads, 33.7 us against 33.3 without all of it, 2 of 3000 + 300, 32/8 heads, 226 against 225.

// x = p[0] + p[1] + p[2] exactly (from 2^-110 on, while x rounds to a finite bf16)
// x - (its bf16 part) is one product of two with a constant, for which no bf16 has to be widened first.  The constants are kept
// out of the compiler's sight: it would encode {-1, 0} as the inline operand -1.0, which the hardware reads as {0, -1}.
struct SplitBy {
    uint32_t low = 0x0000bf80, high = 0xbf800000;  // bf16 pairs {-1, 0} and {0, -1}
    __device__ __forceinline__ SplitBy() { asm volatile("" : "+s"(low), "+s"(high)); }
};
__device__ __forceinline__ void split3(const SplitBy& by, const float* x, bf16x8* p) {
    const bf16x2 kLow = __builtin_bit_cast(bf16x2, by.low), kHigh = __builtin_bit_cast(bf16x2, by.high);
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
        const bf16x2 h = {(__bf16)x[i], (__bf16)x[i + 1]};
        const float r0 = __builtin_amdgcn_fdot2_f32_bf16(h, kLow, x[i], false), r1 = __builtin_amdgcn_fdot2_f32_bf16(h, kHigh, x[i + 1], false);
        const bf16x2 m = {(__bf16)r0, (__bf16)r1};
        const float s0 = __builtin_amdgcn_fdot2_f32_bf16(m, kLow, r0, false), s1 = __builtin_amdgcn_fdot2_f32_bf16(m, kHigh, r1, false);
        const bf16x2 l = {(__bf16)s0, (__bf16)s1};
        p[0][i] = h[0], p[0][i + 1] = h[1];
        p[1][i] = m[0], p[1][i + 1] = m[1];
        p[2][i] = l[0], p[2][i + 1] = l[1];
    }
}

// The least magnitude, and the sum of all (infinite or NaN where one is): both in the vector registers, as a flag per number
// is a vector compare and a scalar or.  With flags the check of Q and of the outputs cost a short call a tenth of its time.
struct Sizes {
    float least = INFINITY, sum = 0.f;
    __device__ __forceinline__ void add(const f32x4& x) {
        least = fminf(fminf(least, fminf(fabsf(x[0]), fabsf(x[1]))), fminf(fabsf(x[2]), fabsf(x[3])));
        sum += (fabsf(x[0]) + fabsf(x[1])) + (fabsf(x[2]) + fabsf(x[3]));
    }
};
template <int N>
__device__ __forceinline__ bool any_tiny(const f32x4* x) {
    uint32_t least = UINT32_MAX;
#pragma unroll
    for (int i = 0; i < N * 4; ++i) least = min(least, __float_as_uint(fabsf(x[i / 4][i % 4])) - 1);  // 0 comes out largest
    return least < __float_as_uint(kTiny) - 1;
}

template <int D, int NW, class Work>
__global__ __launch_bounds__(64 * NW, D == 64 ? 3 : 2) void attn_f32_split_kernel(AttnLaunch a, Work wk) {
    constexpr int TR = kAttnF32SplitRows;
    constexpr int KS = D / 32;         // k-steps of a score
    constexpr int DT = D / 32;         // accumulators of 32 output columns
    constexpr int CPR = D / 4;         // 16-byte chunks per row
    constexpr int ROWB = D * 4;        // bytes per row
    constexpr int PLANEB = KT * ROWB;  // one tile of K (or V)
    constexpr int RPI = 64 / CPR;      // rows one copy instruction covers
    constexpr int NI = KT / RPI;       // copy instructions per plane and tile
    static_assert(TR * ROWB == 2 * PLANEB, "a wave's output fits its tile buffers");
    // the waves' tiles, and behind them Q, later (max, sum) of every wave and row
    __shared__ __attribute__((aligned(1024))) char smem[NW * 2 * PLANEB + TR * ROWB];
    char* const qs = smem + NW * 2 * PLANEB;
    float2(*const MLs)[TR] = reinterpret_cast<float2(*)[TR]>(qs);
    static_assert(NW * TR * 8 + 4 <= TR * ROWB, "states and the flag fit the Q rows");
    typedef volatile __attribute__((address_space(3))) int lds_flag;  // a generic pointer's accesses would wait for the copies
    lds_flag* const flag = (lds_flag*)(qs + TR * ROWB - 4);

    touch_args(a, wk);
    const int Hkv = a.kv_heads;
    int g, entry;
    split_block_id(a, blockIdx.x, &g, &entry);
    entry += wk.entry0;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const WorkItem it = find_item(wk, entry, a.group, TR);
    const int P = it.prefix, N = it.new_len, s0 = it.new_start, G = a.group;
    const uint32_t g_magic = a.group_magic;
    auto div_g = [&](uint32_t x) { return g_magic ? (int)__umulhi(x, g_magic) : (int)x; };  // exact while x * G < 2^32
    const long long row0 = (long long)it.tile * TR;
    const int rows_here = (int)min((long long)TR, (long long)N * G - row0);
    const int tok0 = row0 * G >> 32 ? (int)(row0 / G) : div_g((uint32_t)row0);  // row 0 of the tile: token tok0,
    const int h0 = (int)(row0 - (long long)tok0 * G);                          // head h0 of the group

    const float* __restrict__ q = static_cast<const float*>(a.q);
    const float* __restrict__ k_new = static_cast<const float*>(a.k_new);
    const float* __restrict__ v_new = static_cast<const float*>(a.v_new);
    const float* __restrict__ pool_k = static_cast<const float*>(a.pool_k);
    const float* __restrict__ pool_v = static_cast<const float*>(a.pool_v);
    const int32_t* __restrict__ table = a.block_table + (long long)it.req * a.table_stride;

    const int l16 = lane & 15, kg = lane >> 4, l32 = lane & 31, hf = lane >> 5;
    const int kv_limit = P + tok0 + div_g(h0 + rows_here - 1) + 1;  // keys [0, kv_limit) are visible to some row
    const int ntiles = (kv_limit + KT - 1) / KT;
    const int nsteps = ntiles > w ? (ntiles - w + NW - 1) / NW : 0;  // this wave takes tiles w, w + NW, ...
    const int my_vis = P + tok0 + div_g(h0 + min(l32, rows_here - 1)) + 1;  // of row l32; rows past the end repeat the last one
    const int vis_min = P + tok0 + 1;  // tiles below need no mask

    // block ids of this wave's tiles, 64 steps at a time, one per lane
    int blk_base = 0, blk_vec;

    // Q: every wave needs all rows, so they are copied to LDS once and shared, 1 KiB per instruction
    {
        constexpr int NQ = TR / RPI / NW;
        const void* src[NQ];
#pragma unroll
        for (int x = 0; x < NQ; ++x) {
            const int r = RPI * (w + x * NW) + lane / CPR, row = h0 + min(r, rows_here - 1), tok = div_g(row);
            src[x] = q + ((long long)(s0 + tok0 + tok) * a.q_heads + g * G + (row - tok * G)) * D + ((lane % CPR) ^ (r & 15)) * 4;
        }
        blk_vec = load_ahead_of_copies<NQ>(table + min(w + lane * NW, ntiles - 1), src,
                                           (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)qs + w * 1024, NW * 1024);
    }

    // Copies: lane i of instruction n brings row RPI n + i / CPR of the tile.  K rows (and Q rows) are stored with their
    // chunk index XORed with the row (on the global side), so that the 16 keys of an operand read hit different banks.
    typedef __attribute__((address_space(3))) char lds_char;
    typedef const __attribute__((address_space(3))) f32x4 lds_f32x4;
    lds_char* const kbuf = (lds_char*)smem + w * (2 * PLANEB);
    lds_char* const vbuf = kbuf + PLANEB;
    const uint32_t k_addr = (uint32_t)(uintptr_t)kbuf, v_addr = k_addr + PLANEB;
    const int new_row = Hkv * D;                                    // elements between fresh rows
    const long long new_off = ((long long)(s0 - P) * Hkv + g) * D;  // of the fresh row at position 0
    auto copy_tile = [&](int step, bool is_k) {
        const int base = (w + step * NW) * KT;
        const long long boff = (long long)__builtin_amdgcn_readlane(blk_vec, step - blk_base) * a.block_stride + (long long)g * kBlock * D;
        const float* pool = is_k ? pool_k : pool_v;
        const float* fresh = is_k ? k_new : v_new;
        const uint32_t dst = is_k ? k_addr : v_addr;
        // Lane offsets of instruction n of a plane, less what the instructions' own offsets add.  Held from tile to tile they
        // are 32 registers; the cached rows' are one exclusive or away from that of instruction 0 (K), or all the same (V).
        int l = lane;
        asm volatile("" : "+v"(l));
        const int lane_off = is_k ? l * 16 ^ (l / CPR) << 4 : l * 16;
        auto copy_runs = [&](uint64_t src, auto off_of) {  // four instructions, 4 KiB of LDS, at a time
#pragma unroll
            for (int n0 = 0; n0 < NI; n0 += 4) {
                uint32_t off[4];
#pragma unroll
                for (int n = 0; n < 4; ++n) off[n] = (uint32_t)off_of(n0 + n);
                dma_runs<4>(src + n0 * 1024, off, dst + n0 * 1024);
            }
        };
        if (base + KT <= P) {  // one pool block: uniform base, per-lane constant offset
            copy_runs(uniform_u64(pool + boff), [&](int n) { return is_k ? lane_off ^ (RPI * n) << 4 : lane_off; });
        } else if (base >= P && base + KT <= kv_limit) {  // fresh rows, all inside the horizon
            const int row_off = l / CPR * (new_row * 4 - ROWB), step_off = RPI * new_row * 4 - 1024;
            copy_runs(uniform_u64(fresh + new_off + (long long)base * new_row),
                      [&](int n) { return (is_k ? lane_off ^ (RPI * n) << 4 : lane_off) + row_off + n * step_off; });
        } else {  // the prefix or the horizon ends inside: source per row; keys past the horizon repeat the last visible one
#pragma unroll 1
            for (int n = 0; n < NI; ++n) {
                const int row = RPI * n + l / CPR, chunk = is_k ? (l % CPR) ^ row : l % CPR;
                const int key = base + row;
                const float* src = key < P ? pool + boff + row * D : fresh + new_off + (long long)min(key, kv_limit - 1) * new_row;
                dma_16B_per_lane(src + chunk * 4, dst + n * 1024);
            }
        }
    };
    // the first tile, as soon as its block id is here
    if (nsteps > 0) {
        copy_tile(0, true);
        copy_tile(0, false);
        wait_vmcnt<2 * NI>();  // this wave's part of Q
    } else {
        wait_vmcnt<0>();
    }

    int koff[KS];  // this lane's K reads: chunks 8 j + kg and 8 j + 4 + kg (the latter: address ^ 64) of row l16
#pragma unroll
    for (int j = 0; j < KS; ++j) koff[j] = l16 * ROWB + (((8 * j + kg) ^ l16) << 4);
    auto read_k = [&](lds_char* rows, int j, float* x) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4 v = *reinterpret_cast<lds_f32x4*>(rows + (koff[j] ^ (h * 64)));
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * h + e] = v[e];
        }
    };
    const SplitBy by;
    block_barrier();  // every wave's part of Q has landed
    bf16x8 qp[2][KS][3];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            float x[8];
            read_k((lds_char*)qs + rb * 16 * ROWB, j, x);
            split3(by, x, qp[rb][j]);
        }
    constexpr int OUT = TR * CPR / (64 * NW);  // chunks of Q, and of the output, per thread
    const float sc = a.scale_log2e;
    f32x4 qx[OUT];
#pragma unroll
    for (int u = 0; u < OUT; ++u) qx[u] = *reinterpret_cast<lds_f32x4*>((lds_char*)qs + (tid + u * 64 * NW) * 16);
    block_barrier();  // the Q rows have been read: their place in LDS is free
    if (tid == 0) *flag = 0;
    bool odd;  // this wave has seen what the split does not keep
    {
        Sizes size;
#pragma unroll
        for (int u = 0; u < OUT; ++u) size.add(qx[u]);
        odd = __builtin_amdgcn_ballot_w64(fmaxf(size.sum, 1.f) * sc > 0x1p96f) != 0;
        if (__builtin_amdgcn_ballot_w64(size.least < kTiny) != 0) odd |= __builtin_amdgcn_ballot_w64(any_tiny<OUT>(qx)) != 0;
    }

    f32x16 oacc[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[t][i] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;  // l: this lane's keys only

    auto do_tile = [&](int step, auto more_c) {
        constexpr bool MORE = decltype(more_c)::value;  // another tile follows
        wait_vmcnt<NI>();  // K is here, V may be under way
        // the five small products of a pair apart from the large one: they are summed where their rounding does not count
        f32x4 big[2], low[2];
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) big[rb] = low[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            float x[8];
            bf16x8 kp[3];
            read_k(kbuf, j, x);
            split3(by, x, kp);
#pragma unroll
            for (int n = 0; n < 6; ++n)
#pragma unroll
                for (int rb = 0; rb < 2; ++rb) {
                    f32x4& s = n < 5 ? low[rb] : big[rb];
                    s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kp[kA[n]], qp[rb][j][kB[n]], s, 0, 0, 0);
                }
        }
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) big[rb] += low[rb];
        if (MORE) {
            if (step + 1 - blk_base >= 64) {
                blk_base = step + 1;
                blk_vec = table[min(w + (step + 1 + lane) * NW, ntiles - 1)];
                asm volatile("" ::"v"(blk_vec));  // the wait for this load stays inside the branch
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this tile's K has been read
            copy_tile(step + 1, true);
        }
        // lane (row l16 of half rb, keys 4 kg + i) -> lane (row l32, keys 8 hf + i, 8 hf + 4 + i)
        float s[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(big[0][i]), __float_as_uint(big[1][i]), false, false);
            s[i] = __uint_as_float(r[0]) * sc;
            s[4 + i] = __uint_as_float(r[1]) * sc;
        }
        const int base = (w + step * NW) * KT;
        if (base + KT > vis_min) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (base + hf * 8 + i >= my_vis) s[i] = -INFINITY;
        }
        // the reference exponent of a row is raised only when a score exceeds it by more than 2^8 (or on the
        // row's first visible key); the two lanes of a row keep the same one
        float mx = s[0];
#pragma unroll
        for (int i = 1; i < 8; ++i) mx = fmaxf(mx, s[i]);
        if (__builtin_amdgcn_ballot_w64(mx > m_run + kRaise) != 0) {
            mx = fmaxf(mx, other_half(mx));
            const bool raise = mx > m_run + kRaise;
            const float alpha = raise ? __builtin_amdgcn_exp2f(m_run - mx) : 1.f;  // first visible key: exp2(-inf) = 0
            m_run = raise ? mx : m_run;
            l_run *= alpha;
#pragma unroll
            for (int t = 0; t < DT; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[t][i] *= alpha;
        }
        const float m_sub = m_run == -INFINITY ? 0.f : m_run;  // a row without a visible key yet: exp2(-inf - 0) = 0
        float p[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) p[i] = __builtin_amdgcn_exp2f(s[i] - m_sub) * kLift;
        l_run += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
        bf16x8 pp[3];
        split3(by, p, pp);
        wait_vmcnt<MORE ? NI : 0>();  // V is here, the next K may be under way
        if (!MORE && base + KT > kv_limit) {
            // rows past the horizon hold the last visible V again, which 0 times its probability only takes out while
            // it is finite (the K rows are masked whatever they hold)
            for (int x = lane; x < (base + KT - kv_limit) * CPR; x += 64)
                *reinterpret_cast<__attribute__((address_space(3))) f32x4*>(vbuf + (kv_limit - base) * ROWB + x * 16) = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int u = 0; u < DT / 2; ++u) {
            f32x2 v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                v[i] = *reinterpret_cast<const __attribute__((address_space(3))) f32x2*>(vbuf + (hf * 8 + i) * ROWB + u * 256 + l32 * 8);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                float x[8];
                bf16x8 vp[3];
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = v[i][t];
                split3(by, x, vp);
#pragma unroll
                for (int n = 0; n < 6; ++n)
                    oacc[2 * u + t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vp[kA[n]], pp[kB[n]], oacc[2 * u + t], 0, 0, 0);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this tile's V has been read
        if (MORE) copy_tile(step + 1, false);
    };
    if (nsteps > 0) {
        for (int step = 0; step + 1 < nsteps; ++step) do_tile(step, std::true_type{});
        do_tile(nsteps - 1, std::false_type{});
    }

    // fused append: this workgroup owns the tokens whose first row (head 0 of the group) it holds
    if (a.fused_append) {
        const int tok_lo = tok0 + (h0 != 0), tok_hi = min(N - 1, tok0 + div_g(h0 + TR - 1));
        float* wk_pool = static_cast<float*>(a.pool_k);
        float* wv_pool = static_cast<float*>(a.pool_v);
        for (int idx = tid; idx < (tok_hi - tok_lo + 1) * (D / 4); idx += 64 * NW) {
            const int tok = tok_lo + idx / (D / 4), c4 = idx % (D / 4);
            const int pos = P + tok;
            const long long src = ((long long)(s0 + tok) * Hkv + g) * D + c4 * 4;
            const long long dst = (long long)table[pos >> 4] * a.block_stride + ((long long)g * kBlock + (pos & 15)) * D + c4 * 4;
            *reinterpret_cast<f32x4*>(wk_pool + dst) = *reinterpret_cast<const f32x4*>(k_new + src);
            *reinterpret_cast<f32x4*>(wv_pool + dst) = *reinterpret_cast<const f32x4*>(v_new + src);
        }
    }

    // combine the waves' states (each left in the wave's own part of LDS, [row][chunk of 4 columns], chunks XORed with the
    // row against bank conflicts): out = sum_w O_w 2^(m_w - m) / sum_w l_w 2^(m_w - m)
    l_run += other_half(l_run);
    if (hf == 0) MLs[w][l32] = float2{m_run, l_run};
    auto ochunk = [&](int r, int c4) { return r * ROWB + ((c4 ^ (r & (CPR - 1))) << 4); };
#pragma unroll
    for (int u = 0; u < DT / 2; ++u)
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            const int m = (i >> 2) * 8 + hf * 4 + (i & 3);  // columns 64 u + 2 m ..
            const f32x4 v = {oacc[2 * u][i], oacc[2 * u + 1][i], oacc[2 * u][i + 1], oacc[2 * u + 1][i + 1]};
            *reinterpret_cast<__attribute__((address_space(3))) f32x4*>(kbuf + ochunk(l32, 16 * u + m / 2)) = v;
        }
    __syncthreads();
    float* __restrict__ out = static_cast<float*>(a.out);
    f32x4 res[OUT];
    Sizes size;
#pragma unroll
    for (int u = 0; u < OUT; ++u) {
        const int r = (tid + u * 64 * NW) / CPR, c4 = tid % CPR;
        float2 ml[NW];
        float m = -INFINITY, l = 0.f;
#pragma unroll
        for (int x = 0; x < NW; ++x) {
            ml[x] = MLs[x][r];
            m = fmaxf(m, ml[x].x);
        }
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int x = 0; x < NW; ++x) {
            const float wgt = ml[x].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[x].x - m);  // a wave may have seen no key of the row
            l += ml[x].y * wgt;
            const f32x4 ox = *reinterpret_cast<lds_f32x4*>((lds_char*)smem + x * (2 * PLANEB) + ochunk(r, c4));
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] += ox[e] * wgt;
        }
        const float inv = 1.f / l;
#pragma unroll
        for (int e = 0; e < 4; ++e) res[u][e] = o[e] * inv;
        size.add(res[u]);
    }
    odd |= __builtin_amdgcn_ballot_w64(!(size.sum < INFINITY)) != 0;
    if (__builtin_amdgcn_ballot_w64(size.least < kTiny) != 0) odd |= __builtin_amdgcn_ballot_w64(any_tiny<OUT>(res)) != 0;
    if (odd && lane == 0) *flag = 1;
    block_barrier();
    if (*flag != 0) {
        float(*const Ms)[16] = reinterpret_cast<float(*)[16]>(qs + 16 * ROWB);  // behind 16 rows of Q
#pragma unroll 1
        for (int half = 0; half < 2; ++half) {
            __syncthreads();
            if (2LL * it.tile * 16 + half * 16 < (long long)N * G) plain_rows<D, NW>(a, it, g, 2 * it.tile + half, false, smem, qs, Ms, Ms + NW);
        }
        return;
    }
#pragma unroll
    for (int u = 0; u < OUT; ++u) {
        const int r = (tid + u * 64 * NW) / CPR, c4 = tid % CPR;
        const int dtok = div_g(h0 + r), head = g * G + h0 + r - dtok * G;
        if (r < rows_here) *reinterpret_cast<f32x4*>(out + ((long long)(s0 + tok0 + dtok) * a.q_heads + head) * D + c4 * 4) = res[u];
    }
}

template <int D, int NW, class Work>
void launch_one(const AttnLaunch& a, const Work& wk, int entries, int rows, hipStream_t s) {
    const dim3 grid((unsigned)entries * a.kv_heads), block(64 * NW);
    if (rows == kAttnF32SplitRows) hipLaunchKernelGGL((attn_f32_split_kernel<D, NW, Work>), grid, block, 0, s, a, wk);
    else hipLaunchKernelGGL((attn_f32_kernel<D, NW, Work>), grid, block, 0, s, a, wk);
}
template <class Work>
void launch_list(const AttnLaunch& a, const Work& wk, int entries, int rows, int waves, hipStream_t s) {
    if (waves == 4) a.head_dim == 64 ? launch_one<64, 4>(a, wk, entries, rows, s) : launch_one<128, 4>(a, wk, entries, rows, s);
    else a.head_dim == 64 ? launch_one<64, 8>(a, wk, entries, rows, s) : launch_one<128, 8>(a, wk, entries, rows, s);
}

}  // namespace

hipError_t launch_attn_f32(const AttnLaunch& a, const AttnWork& wk, int entries, int rows, int waves, hipStream_t s) {
    if (entries <= 0) return hipSuccess;
    wk.n_reqs <= kAttnReqStep ? launch_list(a, short_list(wk), entries, rows, waves, s) : launch_list(a, wk, entries, rows, waves, s);
    return hipGetLastError();
}

}  // namespace ragc
