// What the matrix-core GEMMs use on the device: vector types, the LDS address space, compile-time loops, the
// rounding to bf16, the swizzle of row-major stages, direct loads into LDS and the waits for them, the order of tiles and the wait in
// front of the sums.
#pragma once
#include "tf_internal.h"

#include <type_traits>
#include <utility>

namespace tf {
namespace {

constexpr int kXcds = 8;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t U2 __attribute__((ext_vector_type(2)));
typedef uint32_t U4 __attribute__((ext_vector_type(4)));
typedef float F4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x4* LdsBf16x4Ptr;

#define TF_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

// f(integral_constant<int, 0>), ..., f(integral_constant<int, N - 1>), in this order
template <class F, int... I>
__host__ __device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__host__ __device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// two binary32 -> packed bf16, round to nearest even (one v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t f32x2_to_bf16x2(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

// Stages of 128-byte rows (layout kNT): which physical 16-byte chunk of its row holds logical chunk c of tile
// row R: c ^ nt_swizzle(R).  An operand read (ds_read_b128) takes 16 consecutive rows, lane l row l % 16,
// logical chunk l / 16 (+ 4 for the second sub-step).  The LDS serves such a read 16 lanes at a
// time, 8 consecutive lanes together with the 8 lanes 32 further on (counters: with a swizzle that
// only kept 16 consecutive lanes apart, every read took twice its cycles): rows r .. r + 7 of
// chunks q and q ^ 2 must fall into 16 different 16-byte bank groups, and a row's parity already
// selects the half of the banks (row pitch 128 bytes).  Bits 1 and 2 of the row go to bits 0 and 2
// of the swizzle, which the chunk pair does not touch; bit 3 of the row goes to bit 1, which
// also keeps 16 consecutive lanes (one chunk, 16 rows) apart.
__host__ __device__ __forceinline__ constexpr int nt_swizzle(int R) {
    return ((R >> 1) & 1) | (((R >> 3) & 1) << 1) | (((R >> 2) & 1) << 2);
}

typedef U4 U4any __attribute__((aligned(2)));       // a 16-byte piece at any element address

// One direct-to-LDS load: lane i fetches 16 bytes from gbase + voff and the wave's 1 KB lands
// at LDS byte address lds_wave_base + kLdsOff + 16 i (the LDS address goes through M0).
// Written as inline assembly so that the compiler's wait-count insertion does not treat every
// later LDS read as dependent on it (it would drain the load queue before each transpose read);
// completion is awaited explicitly with wait_direct_loads() before the stage barrier.
// The addition sets SCC, and the compiler is free to place the statement between the two
// halves of one of its own 64-bit scalar additions (s_add_u32 / s_addc_u32) unless it is told:
// a clobbered carry sends the high word of a global address off by one as soon as the addition
// crosses a 4 GiB boundary.  Hence the "scc" clobber; the build scans the generated code for
// inline assembly between a producer and a consumer of SCC and refuses it.  M0 is named for the
// same reason: the compiler keeps values of its own there (LDS-DMA builtins, lane selects).
template <int kLdsOff>
__device__ __forceinline__ void direct_load_16B(const char* gbase, uint32_t voff, uint32_t lds_wave_base) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_wave_base), "v"(voff), "s"(gbase), "n"(kLdsOff)
                 : "memory", "scc", "m0");
}
__device__ __forceinline__ void wait_direct_loads() {
    __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0), other counters untouched
}
// vmcnt(n), other counters untouched
template <int n>
__device__ __forceinline__ void wait_loads() {
    static_assert(n < 64, "six bits");
    __builtin_amdgcn_s_waitcnt(0x0f70 | (n & 15) | ((n >> 4) << 14));
}
// All but the `stages` youngest stages of kPer loads, and kAfter loads behind them, have arrived.
template <int kPer, int kMost, int kAfter = 0>
__device__ __forceinline__ void wait_stages(int stages) {
    if (stages >= kMost) wait_loads<kPer * kMost + kAfter>();
    else if constexpr (kMost > 0) wait_stages<kPer, kMost - 1, kAfter>(stages);
}

// Block number -> logical tile of a launch with a block per tile: runs of 8 consecutive tiles stay on one XCD (block b
// runs on XCD b % 8).
__device__ __forceinline__ int logical_tile(int b, int nb) {
    constexpr int kXcdRun = 8, span = kXcds * kXcdRun;
    if (b >= (nb / span) * span) return b;
    const int xcd = b % kXcds, idx = b / kXcds;
    return ((idx / kXcdRun) * kXcds + xcd) * kXcdRun + idx % kXcdRun;
}

// Between the last matrix instruction and the first vector instruction that reads its result.  Left to
// itself the compiler counts a wait and a barrier in between as wait states, and an fp32 sum's last
// register, read first behind the two, was the old one.  The sums pass through statements in front of the
// wait and behind it: no matrix instruction can follow it, no reader precede it.  (The build looks through
// the generated code for a reader that comes too early.)
template <class V, int kI, int kJ>
__device__ __forceinline__ void wait_for_sums(V (&x)[kI][kJ]) {
    auto tie = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kI; ++i)
#pragma unroll
            for (int j = 0; j < kJ; ++j) asm volatile("" : "+v"(x[i][j]));
    };
    tie();
    asm volatile("s_nop 15\n\ts_nop 15");
    tie();
}

}  // namespace
}  // namespace tf
