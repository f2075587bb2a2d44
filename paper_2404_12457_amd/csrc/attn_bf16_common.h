// Device helpers shared by the bf16 attention kernels (gfx950 only).
#pragma once
#include <type_traits>

#include "ragc_internal.h"

namespace ragc {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int TN = 64;                    // keys per LDS tile
constexpr float kRescaleThreshold = 8.f;  // log2 units
constexpr float kRaiseSum = 256.f;        // of a lane's probabilities of a tile
constexpr bf16x2 kOnes2 = {(__bf16)1.0f, (__bf16)1.0f};

// Wave-wide copy of 64 x 16 bytes from global memory straight into LDS: lane i's 16 bytes
// land at lds_addr + 16*i.  Issued as inline assembly on purpose: the compiler's own
// bookkeeping for this instruction drains every outstanding load before the next LDS read,
// which would serialise the copies; the waits are placed by hand (wait_vmcnt, and block_barrier
// where a tile is shared between waves).
// The s_nop is required: the LDS address travels in M0, and a scalar write of M0 needs one wait
// state before an LDS-DMA instruction reads it (inside inline assembly nobody inserts it for us;
// without it the copy can land at the previous instruction's LDS address).
__device__ __forceinline__ void dma_16B_per_lane(const void* gptr, uint32_t lds_addr) {
    lds_addr = __builtin_amdgcn_readfirstlane(lds_addr);  // wave-uniform by construction; make the register class explicit
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(gptr) : "memory", "m0");
}
// N runs of 64 x 16 bytes from a wave-uniform base address: run i comes from sbase + off[i] + OFF0 + 1024 i and lands at
// lds_addr + OFF0 + 1024 i (the instruction's offset counts on both sides, so one write of M0 serves all).  sbase is in scalar
// registers that a vector instruction (a readfirstlane) may have written just before: five wait states before the first load
// reads them.
// No "memory" clobber, so that the compiler may move LDS reads of another buffer across the copies.  Reads of the buffer they
// write cannot come near: the callers put a wait with such a clobber between the last read and the copies (lgkmcnt(0), or
// block_barrier) and another one between the copies and the next read (wait_vmcnt).
template <int N, int OFF0 = 0>
__device__ __forceinline__ void dma_runs(uint64_t sbase, const uint32_t* off, uint32_t lds_addr) {
    static_assert((N == 2 || N == 4) && OFF0 + (N - 1) * 1024 < 4096, "offset field");
    if constexpr (N == 2)
        asm volatile(
            "s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %3 offset:%4\n\tglobal_load_lds_dwordx4 %2, %3 offset:%5"
            ::"s"(lds_addr), "v"(off[0]), "v"(off[1]), "s"(sbase), "n"(OFF0), "n"(OFF0 + 1024)
            : "m0");
    else
        asm volatile(
            "s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %5 offset:%6\n\tglobal_load_lds_dwordx4 %2, %5 offset:%7\n\t"
            "global_load_lds_dwordx4 %3, %5 offset:%8\n\tglobal_load_lds_dwordx4 %4, %5 offset:%9"
            ::"s"(lds_addr), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(sbase), "n"(OFF0), "n"(OFF0 + 1024),
              "n"(OFF0 + 2048), "n"(OFF0 + 3072)
            : "m0");
}
// One dword per lane from `p`, and behind it N copies of 64 x 16 bytes straight into LDS (lane i's from src[x], to lds_addr +
// x * stride + 16 i); returns when the dword is here, with the copies still under way.  All in one statement: the load's
// register is not the compiler's before it has been written, and the compiler's own wait for it would drain the copies.
template <int N>
__device__ __forceinline__ int load_ahead_of_copies(const int32_t* p, const void* const* src, uint32_t lds_addr, uint32_t stride) {
    static_assert(N == 1 || N == 2 || N == 4, "copies");
    int v;
    lds_addr = __builtin_amdgcn_readfirstlane(lds_addr);
    if constexpr (N == 1)
        asm volatile("global_load_dword %0, %1, off\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, off\n\ts_waitcnt vmcnt(1)"
                     : "=&v"(v) : "v"(p), "s"(lds_addr), "v"(src[0]) : "memory", "m0");
    else if constexpr (N == 2)
        asm volatile(
            "global_load_dword %0, %1, off\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %4, off\n\t"
            "s_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %5, off\n\ts_waitcnt vmcnt(2)"
            : "=&v"(v) : "v"(p), "s"(lds_addr), "s"(lds_addr + stride), "v"(src[0]), "v"(src[1]) : "memory", "m0");
    else
        asm volatile(
            "global_load_dword %0, %1, off\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %6, off\n\t"
            "s_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %7, off\n\ts_mov_b32 m0, %4\n\ts_nop 0\n\t"
            "global_load_lds_dwordx4 %8, off\n\ts_mov_b32 m0, %5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %9, off\n\ts_waitcnt vmcnt(4)"
            : "=&v"(v) : "v"(p), "s"(lds_addr), "s"(lds_addr + stride), "s"(lds_addr + 2 * stride), "s"(lds_addr + 3 * stride),
              "v"(src[0]), "v"(src[1]), "v"(src[2]), "v"(src[3]) : "memory", "m0");
    return v;
}
__device__ __forceinline__ uint64_t uniform_u64(const void* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ float other_half(float x) {
    // value held by lane ^ 32
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
}

__device__ __forceinline__ float other_quarter(float x) {
    // value held by lane ^ 16
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float((threadIdx.x & 16) ? r[0] : r[1]);
}

// XOR pattern applied to the 16-byte chunk index of row `row` (depends on row & 15), for operands of 64 / KG rows; KG = 4 at
// head_dim 128 only.
// KG = 2 (v_mfma_f32_32x32x16_bf16): an operand read takes one chunk of 32 rows, a transposing read four of every fourth.
// KG = 4 (16x16x32): an operand read takes four chunks of 16 rows, lanes 0-3, 12-15 and 20-27 at a time (or the others of 32),
// a transposing read two chunks of rows 0-7 or 8-15.  Both without bank conflicts: 64 KiB in 280 cycles per CU.
template <int D, int KG = 2>
__device__ __forceinline__ int swz(int row) {
    static_assert(KG == 2 || (KG == 4 && D == 128), "swizzle");
    if (KG == 4) {
        const int b2 = (row >> 2) & 1, b3 = (row >> 3) & 1;
        return ((row & 3) << 2) | ((b2 ^ b3) << 1) | b3;
    }
    if (D == 128) return ((row & 3) << 2) | ((row >> 2) & 3);
    return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
}

// wait until at most N vector-memory operations of this wave are outstanding
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

__device__ __forceinline__ void block_barrier() {
    // hardware barrier without the fence of __syncthreads(): outstanding LDS-DMA loads of
    // later tiles must stay in flight across it
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}


}  // namespace
}  // namespace ragc
