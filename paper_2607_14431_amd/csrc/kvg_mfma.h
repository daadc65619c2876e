// Device helpers shared by the MFMA kernels: operand types, half swaps, buffer resources, fp8
// widening.
#pragma once

#include "kvg_device.h"

#include <math.h>

namespace kvg {

namespace {

// A lane's value and that of lane ^ 32, as (the value in lanes 0-31, the value in lanes
// 32-63): both halves of the wave get the same pair, so a reduction of the two is the same
// bits in both.  A VALU half swap, where a cross-lane shuffle would be an LDS round trip whose
// wait also drains every LDS read issued before it.
__device__ inline float2 halves32(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return make_float2(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
typedef __attribute__((address_space(3))) char lds_char;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) u32x2 lds_u32x2;
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) i32x2 lds_i32x2;

// Fourth word of a raw buffer resource on gfx9-family targets (32-bit data format, no
// swizzle): accesses past num_records return zeros instead of touching memory.
constexpr int kBufferWord3 = 0x00020000;

__device__ __forceinline__ bf16x8 as_bf16x8(const uint4& v) { return __builtin_bit_cast(bf16x8, v); }

// two fp32 -> packed bf16, round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16_rne(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){lo, hi}, bf16x2));
}

// whether every element is a finite number (0 x is 0 for those alone)
template <int N>
__device__ __forceinline__ bool all_finite(const f32x16 (&o)[N]) {
  float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int d = 0; d < N; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r % 4] = fmaf(o[d][r], 0.0f, z[r % 4]);
  const float sum = (z[0] + z[1]) + (z[2] + z[3]);
  return sum == 0.0f;
}

// eight fp8 values (two words) -> eight bf16 values, exactly
__device__ __forceinline__ uint4 widen_fp8x8(uint32_t lo, uint32_t hi) {
  return make_uint4(__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)lo, 1.0f, false)),
                    __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)lo, 1.0f, true)),
                    __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)hi, 1.0f, false)),
                    __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)hi, 1.0f, true)));
}

}  // namespace

}  // namespace kvg
