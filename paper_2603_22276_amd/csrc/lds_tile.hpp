// Building blocks the matrix-core kernels share: swizzled LDS layouts, fragment reads, waits.
#pragma once

#include "common.hpp"

#include <type_traits>
#include <utility>

namespace dora {
namespace {

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));
typedef uint64_t u64x1_t;
typedef uint64_t u64x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void* lds_void_ptr_t;

// The LDS serves a 16-byte-per-lane access 16 lanes at a time, and those 16 lanes must touch 16
// different 16-byte slots modulo 256 bytes.
//
// K-contiguous operand: [rows][64] bf16, 128 bytes per row, the chunk index XORed with row/2: the 16
// rows one group of lanes reads (same logical chunk) then cover all 16 slots.
template <int BK>
__device__ __forceinline__ int kc_swizzle(int row)
{
    static_assert(BK == 64, "swizzle of 128-byte rows");
    return (row >> 1) & 7;
}
template <int BK>
__device__ __forceinline__ int lds_off(int row, int k)
{
    return row * (BK * 2) + ((((k >> 3) ^ kc_swizzle<BK>(row)) & (BK / 8 - 1)) << 4) + ((k & 7) << 1);
}
// K-strided operand: kept as loaded, [BK][ROWS] bf16; chunks of 8 rows XORed with 4*(k mod 4) so the four
// k-rows one transposing read touches fall into different slots, and with 2*(bit 3 of k) so that two
// 16-lane blocks reading the same rows 8 k-rows apart do too.
__device__ __forceinline__ int ks_swizzle(int k)
{
    return ((k & 3) << 2) | (((k >> 3) & 1) << 1);
}
template <int ROWS>
__device__ __forceinline__ int lds_off_ks(int row, int k)
{
    static_assert(ROWS >= 128, "swizzle needs at least 16 chunks per k-row");
    return k * (ROWS * 2) + ((((row >> 3) ^ ks_swizzle(k))) << 4) + ((row & 7) << 1);
}

// Compile-time loop: f(std::integral_constant<int, 0>{}), ..., f(std::integral_constant<int, N - 1>{})
template <class F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// LDS reads are issued as inline assembly with immediate offsets: the compiler neither tracks them in
// lgkmcnt nor makes them wait for global -> LDS loads still in flight to other ring slots, so every
// consumer is preceded by an explicit wait_lgkmcnt.
template <int OFF>
__device__ __forceinline__ bf16x8_t lds_read_b128(uint32_t addr)
{
    static_assert(OFF >= 0 && OFF < 65536, "ds_read offset field is 16 bits");
    bf16x8_t v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
// Two transposing reads (k and k + 4 of a K-strided tile, HI bytes apart) forming one MFMA fragment.
// ds_read_b64_tr_b16: inside each block of 16 lanes, lane i receives element (i & 3) of the 8 bytes
// addressed by lanes i/4, i/4 + 4, i/4 + 8, i/4 + 12.
template <int OFF, int HI>
__device__ __forceinline__ bf16x8_t lds_read_tr(uint32_t addr)
{
    static_assert(OFF >= 0 && OFF + HI < 65536, "ds_read offset field is 16 bits");
    u64x1_t lo, hi;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(addr), "n"(OFF));
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(addr), "n"(OFF + HI));
    u64x2_t v = {lo, hi};
    return __builtin_bit_cast(bf16x8_t, v);
}

// Byte offset, inside an operand's LDS tile, that lane `lane` reads for the MFMA fragment of the 32
// rows starting at row0: the lane gets row row0 + (lane & 31), k = k16*16 + 8*(lane >> 5) + 0..7.
// K-contiguous tile: one 16-byte read.  K-strided tile: the lane points at k-row
// k16*16 + 8*(lane >> 5) + (lane & 15) / 4 and rows 4*(lane & 3) .. +3 of its 16-lane block; blocks 1
// and 3 sit 16 rows further; the second read takes k + 4 (same swizzle).
template <int ROWS, int BK, bool KCONTIG>
__device__ __forceinline__ uint32_t frag_off(int row0, int k16, int lane)
{
    if (KCONTIG) return (uint32_t)lds_off<BK>(row0 + (lane & 31), k16 * 16 + (lane >> 5) * 8);
    return (uint32_t)lds_off_ks<ROWS>(row0 + ((lane >> 4) & 1) * 16 + (lane & 3) * 4,
                                      k16 * 16 + (lane >> 5) * 8 + ((lane & 15) >> 2));
}

// The same for the 16x16x32 MFMA: the lane gets row row0 + (lane & 15), k = k32*32 + 8*(lane >> 4) + 0..7.
// K-strided tile: the lane points at k-row k32*32 + 8*(lane >> 4) + (lane & 15) / 4 and rows 4*(lane & 3) .. +3.
template <int ROWS, int BK, bool KCONTIG>
__device__ __forceinline__ uint32_t frag16_off(int row0, int k32, int lane)
{
    if (KCONTIG) return (uint32_t)lds_off<BK>(row0 + (lane & 15), k32 * 32 + (lane >> 4) * 8);
    return (uint32_t)lds_off_ks<ROWS>(row0 + (lane & 3) * 4, k32 * 32 + (lane >> 4) * 8 + ((lane & 15) >> 2));
}

// s_waitcnt with only one counter constrained (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt
// 6:4, lgkmcnt 11:8; the others are left at their maxima)
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N <= 63, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}
template <int N>
__device__ __forceinline__ void wait_lgkmcnt()
{
    static_assert(N >= 0 && N <= 15, "lgkmcnt is a 4-bit counter");
    __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));
}

}  // namespace
}  // namespace dora
