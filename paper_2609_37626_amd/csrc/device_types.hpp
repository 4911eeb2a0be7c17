// Vector types and small conversions that the gfx950 kernels share.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#define LDS_AS __attribute__((address_space(3)))

namespace splash {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short i16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned pack_bf16x2(float a, float b) {
  bf16x2 v = __builtin_convertvector((f32x2){a, b}, bf16x2);
  return __builtin_bit_cast(unsigned, v);
}
__device__ __forceinline__ unsigned pack_f16x2(float a, float b) {
  f16x2 v = __builtin_convertvector((f32x2){a, b}, f16x2);
  return __builtin_bit_cast(unsigned, v);
}

// Split partials are stored in fp16, each (slot, head) quarter of 128
// columns multiplied by 2^-e: e = 0 unless the quarter's largest magnitude
// m reaches 2^15, else e = floor(log2 m) - 14, so every stored value stays
// below 2^15 and rescales exactly.  The exponent of magnitude m is read from
// its bits (a zero m gives e = 0; e <= 114).
__device__ __forceinline__ uint32_t partial_exponent(float m) {
  const int32_t ex = (int32_t)((__builtin_bit_cast(uint32_t, m) >> 23) & 255u) - 127 - 14;
  return ex > 0 ? (uint32_t)ex : 0u;
}
// Four stored fp16 values (two dwords) back to fp32, times 2^e.
__device__ __forceinline__ f32x4 unpack_f16x4(uint32_t lo, uint32_t hi, int e) {
  const f32x2 a = __builtin_convertvector(__builtin_bit_cast(f16x2, lo), f32x2);
  const f32x2 b = __builtin_convertvector(__builtin_bit_cast(f16x2, hi), f32x2);
  return (f32x4){__builtin_amdgcn_ldexpf(a[0], e), __builtin_amdgcn_ldexpf(a[1], e), __builtin_amdgcn_ldexpf(b[0], e),
                 __builtin_amdgcn_ldexpf(b[1], e)};
}

// f(integral_constant<0>), ..., f(integral_constant<N - 1>)
template <int N, typename F, int... I>
__device__ __forceinline__ void static_for_impl(F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl<N>(f, std::make_integer_sequence<int, N>{});
}

}  // namespace splash
