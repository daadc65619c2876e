// KV-append: fresh computation of new tokens' keys/values into the paged cache, plus the
// rotated queries the attention kernels read.
//
// One workgroup per (sequence, new token) and group of layers.  The token's absolute
// position is the same for every layer and head, so the workgroup computes the D/2
// angles pos * theta_i in fp64 once, takes cos/sin in fp64, rounds them to fp32 into
// LDS, and every thread then rotates 16-byte vectors of its rows with the fixed fp32
// formula of rotate_pair().  Keys are rounded to the storage dtype (nearest even) and
// written through the block table; values are copied (rounded to fp8 for an fp8 cache,
// whose raw inputs are bf16); queries go to the workspace.
#include "kvg_device.h"
#include "kvg_launch.h"

#include <type_traits>

namespace kvg {

namespace {

// Raw rows are read once and cache rows written once: streaming (nontemporal) accesses
// (the 4,096-token 12B-class prefix: 693 -> 670 us).
typedef unsigned int u32x4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld16(const void* p) {
  const u32x4v v = __builtin_nontemporal_load(reinterpret_cast<const u32x4v*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st16(void* p, const uint4& v) {
  const u32x4v t = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(t, reinterpret_cast<u32x4v*>(p));
}

// Rotated pair values of one item: half pairing reads vectors at element offsets e0 and
// e0 + D/2 (E pairs); interleaved reads one vector (E/2 pairs).
template <typename T>
struct RotItem {
  static constexpr int E = Elem<T>::kPerVec;
  float x[2][E];   // [0]: vector at e0, [1]: partner vector (half pairing only)
};

// An item's raw vectors: at e0, and at e0 + D/2 (half pairing only).
struct RawItem {
  uint4 a, b;
};

template <typename T>
__device__ __forceinline__ RawItem load_item(const T* row, int e0, int half, int pairing) {
  RawItem it;
  it.a = ld16(row + e0);
  it.b = pairing == 0 ? ld16(row + e0 + half) : make_uint4(0, 0, 0, 0);
  return it;
}

template <typename T>
__device__ __forceinline__ void rotate_item(const RawItem& raw, int e0, int pairing, const float* cs, RotItem<T>& it) {
  constexpr int E = Elem<T>::kPerVec;
  if (pairing == 0) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      float a = Elem<T>::get(raw.a, e), b = Elem<T>::get(raw.b, e);
      const int p = e0 + e;
      rotate_pair(a, b, cs[2 * p], cs[2 * p + 1]);
      it.x[0][e] = a;
      it.x[1][e] = b;
    }
  } else {
#pragma unroll
    for (int e = 0; e < E; e += 2) {
      float a = Elem<T>::get(raw.a, e), b = Elem<T>::get(raw.a, e + 1);
      const int p = (e0 + e) >> 1;
      rotate_pair(a, b, cs[2 * p], cs[2 * p + 1]);
      it.x[0][e] = a;
      it.x[0][e + 1] = b;
    }
  }
}

// E consecutive values stored in type T (16 bytes, or 8 for fp8 from a bf16 item)
template <typename T, int E>
__device__ __forceinline__ void store_elems(T* dst, const float* x) {
  uint32_t w[4];
  pack_words<T, E>(x, w);
  if constexpr (E * sizeof(T) == 16)
    st16(dst, make_uint4(w[0], w[1], w[2], w[3]));
  else
    *reinterpret_cast<uint2*>(dst) = make_uint2(w[0], w[1]);
}

// E (8) fp32 values as bf16 hi and lo parts (split_bf16), one 16-byte vector each
template <int E>
__device__ __forceinline__ void store_split(uint16_t* hi, uint16_t* lo, const float* x) {
  static_assert(E == 8, "one 16-byte vector of bf16");
  uint32_t h[E], l[E];
#pragma unroll
  for (int e = 0; e < E; ++e) split_bf16(x[e], h[e], l[e]);
  st16(hi, make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)));
  st16(lo, make_uint4(l[0] | (l[1] << 16), l[2] | (l[3] << 16), l[4] | (l[5] << 16), l[6] | (l[7] << 16)));
}

template <typename T>
__device__ __forceinline__ void store_vec_f32(float* dst, const float* x) {
  constexpr int E = Elem<T>::kPerVec;
#pragma unroll
  for (int e = 0; e < E; e += 4) st16(dst + e, make_uint4(__float_as_uint(x[e]), __float_as_uint(x[e + 1]),
                                                           __float_as_uint(x[e + 2]), __float_as_uint(x[e + 3])));
}

// kAhead: a thread's first item of each kind is requested together with the others' (see below).
template <typename T, bool kAhead>
__global__ __launch_bounds__(256) void append_kernel(const AppendArgs a) {
  using R = typename RawOf<T>::type;                     // raw input type
  constexpr int E = Elem<R>::kPerVec;                    // elements per item vector
  const int tok = blockIdx.x;
  const int b = tok / a.chunk;
  const int i = tok - b * a.chunk;
  const int ctx = a.ctx_lens[b];
  if (ctx < 0 || ctx > a.max_ctx_len) return;           // uniform: bad metadata, skip
  const int t = ctx + i;                                 // < max_pages * kPage (host check)
  const int32_t page = a.block_tables[(int64_t)b * a.max_pages + t / kPage];
  const bool page_ok = page >= 0 && page < a.n_pages;
  const int64_t pos = a.start_pos[b] + t;
  const int D = a.D, half = D >> 1;

  const int items_per_row = (a.pairing == 0) ? (half / E) : (D / E);
  const int vec_per_row = D / E;
  const int n_k = page_ok ? a.Hkv * items_per_row : 0, n_v = page_ok ? a.Hkv * vec_per_row : 0;
  const int n_q = a.q_raw != nullptr ? a.Hq * items_per_row : 0;
  const int l_begin = blockIdx.y * a.layers_per_block;
  const int l_end = min(l_begin + a.layers_per_block, a.n_layers);
  const int row = t % kPage;

  auto raw_tok = [&](int l) -> int64_t { return ((int64_t)l * a.batch + b) * a.chunk + i; };
  auto load_rot = [&](const void* raw, int n_heads, int l, int it) {
    const int h = it / items_per_row;
    return load_item<R>(reinterpret_cast<const R*>(raw) + (raw_tok(l) * n_heads + h) * D, (it - h * items_per_row) * E, half,
                        a.pairing);
  };
  auto load_v = [&](int l, int it) {
    return ld16(reinterpret_cast<const R*>(a.v_raw) + raw_tok(l) * a.Hkv * D + it * E);
  };
  // A thread's first item of each kind, requested together and before the layer's stores, the first
  // layer's before the angles: each kind waiting for its own loads took 10 us of a 512-row chunk
  // with 16 + 8 + 8 heads x 256 instead of 7, and 630 instead of 617 of a 3,950-token block's 48 layers.  Requesting
  // the next layer's ahead of this one's stores costs registers and with them wavefronts: 641.  The first
  // items alone cost two wavefronts of eight a SIMD, which is more than they give where a token has few
  // (launch_append_t).
  struct First {
    RawItem k, q;
    uint4 v;
  };
  const int t0 = threadIdx.x;
  auto fetch = [&](int l) {
    First f{};
    if (t0 < n_k) f.k = load_rot(a.k_raw, a.Hkv, l, t0);
    if (t0 < n_v) f.v = load_v(l, t0);
    if (t0 < n_q) f.q = load_rot(a.q_raw, a.Hq, l, t0);
    return f;
  };
  First cur;
  if constexpr (kAhead) cur = fetch(l_begin);

  __shared__ float cs[2 * kMaxHalfDim];
  for (int p = threadIdx.x; p < half; p += blockDim.x) {
    double s, c;
    sincos((double)pos * a.theta[p], &s, &c);
    cs[2 * p] = (float)c;
    cs[2 * p + 1] = (float)s;
  }
  __syncthreads();

  for (int l = l_begin; l < l_end; ++l) {
    const int64_t lbase = (int64_t)(a.layer0 + l) * a.layer_elems;
    T* kpool = reinterpret_cast<T*>(a.k_pool) + lbase;
    T* vpool = reinterpret_cast<T*>(a.v_pool) + lbase;

    // keys: rotate, round, store through the block table
    for (int it = t0; it < n_k; it += blockDim.x) {
      const RawItem raw = kAhead && it == t0 ? cur.k : load_rot(a.k_raw, a.Hkv, l, it);
      const int h = it / items_per_row;
      const int e0 = (it - h * items_per_row) * E;
      RotItem<R> r;
      rotate_item<R>(raw, e0, a.pairing, cs, r);
      T* dst = kpool + (((int64_t)page * a.Hkv + h) * kPage + row) * D;
      store_elems<T, E>(dst + e0, r.x[0]);
      if (a.pairing == 0) store_elems<T, E>(dst + e0 + half, r.x[1]);
    }
    // values: copy (rounded to the storage type when it differs from the raw type)
    for (int it = t0; it < n_v; it += blockDim.x) {
      const uint4 raw = kAhead && it == t0 ? cur.v : load_v(l, it);
      const int h = it / vec_per_row;
      const int e0 = (it - h * vec_per_row) * E;
      T* dst = vpool + (((int64_t)page * a.Hkv + h) * kPage + row) * D + e0;
      if constexpr (std::is_same<T, R>::value) {
        st16(dst, raw);
      } else {
        float x[E];
#pragma unroll
        for (int e = 0; e < E; ++e) x[e] = Elem<R>::get(raw, e);
        store_elems<T, E>(dst, x);
      }
    }
    for (int it = t0; it < n_q; it += blockDim.x) {
      const RawItem raw = kAhead && it == t0 ? cur.q : load_rot(a.q_raw, a.Hq, l, it);
      const int h = it / items_per_row;
      const int e0 = (it - h * items_per_row) * E;
      RotItem<R> r;
      rotate_item<R>(raw, e0, a.pairing, cs, r);
      const int64_t qoff = (raw_tok(l) * a.Hq + h) * D;
      if constexpr (sizeof(R) == 2) {
        if (a.q_out_bf16) {                        // bf16 hi + lo queries (bf16 and fp8 caches)
          uint16_t* qh = reinterpret_cast<uint16_t*>(a.q_out) + qoff;
          uint16_t* ql = reinterpret_cast<uint16_t*>(a.q_out_lo) + qoff;
          store_split<E>(qh + e0, ql + e0, r.x[0]);
          if (a.pairing == 0) store_split<E>(qh + e0 + half, ql + e0 + half, r.x[1]);
          continue;
        }
      }
      float* q = reinterpret_cast<float*>(a.q_out) + qoff;
      store_vec_f32<R>(q + e0, r.x[0]);
      if (a.pairing == 0) store_vec_f32<R>(q + e0 + half, r.x[1]);
    }
    if constexpr (kAhead) {
      if (l + 1 < l_end) cur = fetch(l + 1);
    }
  }
}

}  // namespace

// kAhead with the queries of a prefill, and from 129 16-byte vectors of values a token on.  48 layers of 1,000 tokens,
// us with / without: fp32, 2 heads x 64 (32 vectors) 48 / 43; bf16, 8 x 64 (64) 64 / 57, 8 x 256 (256) 147 / 149.
template <typename T>
void launch_append_t(const AppendArgs& a, hipStream_t stream) {
  const dim3 grid(a.batch * a.chunk, (a.n_layers + a.layers_per_block - 1) / a.layers_per_block);
  if (a.q_raw != nullptr || a.Hkv * a.D > 128 * Elem<typename RawOf<T>::type>::kPerVec)
    append_kernel<T, true><<<grid, 256, 0, stream>>>(a);
  else
    append_kernel<T, false><<<grid, 256, 0, stream>>>(a);
}

hipError_t launch_append(const AppendArgs& a, int dtype, hipStream_t stream) {
  switch (dtype) {
    case kDtypeF32: launch_append_t<float>(a, stream); break;
    case kDtypeBf16: launch_append_t<uint16_t>(a, stream); break;
    case kDtypeFp8: launch_append_t<uint8_t>(a, stream); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace kvg
