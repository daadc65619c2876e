// Device helpers of the attention kernels: 16-byte row accesses, the rotation and rounding of raw
// rows, merge factors of softmax states.
#pragma once

#include "kvg_device.h"

#include <math.h>

namespace kvg {

namespace {

__device__ __forceinline__ uint4 ld16(const void* p) { return *reinterpret_cast<const uint4*>(p); }
__device__ __forceinline__ void st16(void* p, const uint4& v) { *reinterpret_cast<uint4*>(p) = v; }

// Merge factor exp2(m_part - m_new); a part that saw no key has m = -inf and weight 0.
__device__ __forceinline__ float merge_factor(float m_part, float m_new) {
  return (m_part == -INFINITY) ? 0.0f : exp2f(m_part - m_new);
}

template <typename T>
__device__ __forceinline__ void rotate_chunk(const uint4& va, const uint4& vb, bool first_half, int pair0,
                                             int pairing, const float* cs, float* out) {
  constexpr int E = Elem<T>::kPerVec;
  if (pairing == 0) {
    // va: this chunk, vb: its partner D/2 away; pair index pair0 + e
#pragma unroll
    for (int e = 0; e < E; ++e) {
      float x = first_half ? Elem<T>::get(va, e) : Elem<T>::get(vb, e);   // first-half element
      float y = first_half ? Elem<T>::get(vb, e) : Elem<T>::get(va, e);   // second-half element
      rotate_pair(x, y, cs[2 * (pair0 + e)], cs[2 * (pair0 + e) + 1]);
      out[e] = first_half ? x : y;
    }
  } else {
#pragma unroll
    for (int e = 0; e < E; e += 2) {
      float x = Elem<T>::get(va, e), y = Elem<T>::get(va, e + 1);
      const int p = pair0 + (e >> 1);
      rotate_pair(x, y, cs[2 * p], cs[2 * p + 1]);
      out[e] = x;
      out[e + 1] = y;
    }
  }
}

// Chunk c of an fp32 row, rotated if asked.
template <int D>
__device__ __forceinline__ uint4 storage_chunk(const float* raw_row, int c, bool rotate, int pairing, const float* cs) {
  constexpr int NCH = D / 4;
  const uint4 va = ld16(raw_row + c * 4);
  if (!rotate) return va;
  float x[4];
  if (pairing == 0) {
    const bool first = c < NCH / 2;
    const int cp = first ? c + NCH / 2 : c - NCH / 2;
    rotate_chunk<float>(va, ld16(raw_row + cp * 4), first, (first ? c : cp) * 4, 0, cs, x);
  } else {
    rotate_chunk<float>(va, va, true, c * 2, 1, cs, x);
  }
  return make_uint4(__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3]));
}

}  // namespace

}  // namespace kvg
