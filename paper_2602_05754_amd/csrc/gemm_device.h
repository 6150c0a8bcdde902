// What both matrix-core GEMMs use on the device: vector types, the LDS address space, compile-time loops, the
// rounding to bf16 and the swizzle of row-major stages.
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
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
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

}  // namespace
}  // namespace tf
