// Chunked-prefill attention of fp32 caches on v_mfma_f32_32x32x2_f32: fp32 operands, products and
// sums, so the results are as exact as on the vector ALUs.
//
// Workgroup = (layer, sequence, KV head g, tile, split): a tile is 32 (row, query head) pairs of the
// chunk, heads fastest; a split is kSplit keys at an absolute multiple of 512, so a row's bytes
// do not depend on how its sequence was chunked.  Each of the four waves takes 128 of the split's
// keys in blocks of 32; their states are folded in order in LDS, and the splits by
// prefill_segments_kernel.  In a small call (solo) a workgroup takes a unit of 128 keys, a block a wave, and
// prefill_f32_units_kernel folds a split's units as the waves' states are folded.
//
//   S^T = K Q^T    C = 32 keys x 32 pairs.  A lane's operand of a step is one float of key lane % 32
//                  (of pair lane % 32): step (j, e) takes dims 8 j + e (lanes 0-31) and 8 j + 4 + e
//                  (lanes 32-63), so one 16-byte load feeds four steps.  Four accumulation
//                  chains (j mod 4), added pairwise: shorter chains round less, and independent
//                  ones issue back to back.
//   softmax        per block, against the block's largest score, all fp32; the block's state is folded into
//                  the wave's, so a block's 32 keys are summed alike whichever wave takes them.
//   O^T += V^T P^T step r takes the keys whose weights accumulator element r holds (8 (r / 4) + r % 4,
//                  lanes 32-63 four further), so P is the operand as it stands; V^T block db is
//                  dims ND i + db of lane i, so a lane's ND values are consecutive.
//
// What bounds it: the matrix cores (64 cycles a step); V comes from L2 straight into
// registers, a few loads ahead, K through LDS up to head_dim 128 (V through LDS too would leave one workgroup
// a CU).  4 layers x 2 x 256 rows x 4 heads over 1k keys, head_dim 64: 169 us a pass on the vector ALUs, where
// every row read all its keys again; 70 here, 57 of them this kernel; 512 rows over 4k keys, 8 KV heads x
// 256: 4,627 -> 698.  A few rows over many keys cost more than there, because most of a tile's 32 pairs are padding:
// one row over 8k keys 21 -> 24 us at head_dim 64 (2 KV heads), 38 -> 58 at 256 (8), 4 layers x 4 such rows 31 -> 38 and
// 333 -> 547.  Small calls take prefill_f32_narrow_kernel.
#include "kvg_launch.h"
#include "kvg_mfma.h"
#include "kvg_rows.h"

#include <float.h>
#include <math.h>

#include <type_traits>

namespace kvg {

namespace {

constexpr int kWaves = kF32Units;
constexpr int kUnitKeys = kSplit / kF32Units;

template <int N>
struct FloatVec {
  float x[N];
};

__device__ __forceinline__ FloatVec<8> load8(const float* p) {
  const FloatVec<4> a = __builtin_bit_cast(FloatVec<4>, ld16(p)), b = __builtin_bit_cast(FloatVec<4>, ld16(p + 4));
  return {{a.x[0], a.x[1], a.x[2], a.x[3], b.x[0], b.x[1], b.x[2], b.x[3]}};
}

// tiles of P (row, query head) pairs of a sequence and KV head
__host__ __device__ inline int narrow_tiles(const PrefillArgs& a, int P) { return (int)(((int64_t)a.chunk * a.group + P - 1) / P); }

// Workgroup blockIdx.x of a grid of (tile, slot, KV head, sequence, layer), the tile fastest.  32-bit divisions: the
// code of 64-bit ones is longer than the rest of a small kernel, and a small call waits for its code.
struct F32Item {
  int tile, slot, g, b, l;
};
__device__ __forceinline__ F32Item f32_item(const PrefillArgs& a, uint32_t n_tiles, uint32_t n_slots) {
  uint32_t id = blockIdx.x;
  F32Item it;
  it.tile = (int)(id % n_tiles);
  id /= n_tiles;
  it.slot = (int)(id % n_slots);
  id /= n_slots;
  it.g = (int)(id % (uint32_t)a.Hkv);
  id /= (uint32_t)a.Hkv;
  it.b = (int)(id % (uint32_t)a.batch);
  it.l = (int)(id / (uint32_t)a.batch);
  return it;
}

// v f_v + x f_x, rounded alike wherever states are folded
__device__ __forceinline__ float fold(float v, float f_v, float x, float f_x) { return fmaf(x, f_x, v * f_v); }

// a key's weight in its block, whose reference is m_ref
__device__ __forceinline__ float block_weight(float score, float scale_log2, float m_ref) {
  return __builtin_amdgcn_exp2f(fmaf(score, scale_log2, -m_ref));
}

// Folds the state (pm, pl, pv) of the keys that follow into (m, l, v); (-inf, 0, 0) is the empty one.
__device__ __forceinline__ void fold_state(float& m, float& l, float& v, float pm, float pl, float pv) {
  const float m_new = fmaxf(m, pm), f = merge_factor(m, m_new), pf = merge_factor(pm, m_new);
  l = fold(l, f, pl, pf);
  v = fold(v, f, pv, pf);
  m = m_new;
}

template <int D, bool kSolo>
__global__ __launch_bounds__(64 * kWaves) void prefill_f32_kernel(const PrefillArgs a) {
  constexpr int NJ = D / 8;            // 16-byte K loads per block and lane
  constexpr int ND = D / 32;           // O blocks
  constexpr int NB = ND < 4 ? ND : 4;  // O blocks of a pass over the block's V
  constexpr int LK = 8;                // K loads ahead
  constexpr int LV = 8;                // V loads ahead
  // up to head_dim 128 K blocks of the waves, above it the queries; after the last block the waves' O
  constexpr bool kStaged = D <= 128;
  constexpr int RB = D * 4, NCH = RB / 16;
  constexpr int kOBytes = kWaves * 32 * (D + 1) * 4, kKBytes = kStaged ? kWaves * 32 * RB : 32 * RB;
  __shared__ __attribute__((aligned(1024))) char s_mem[kOBytes > kKBytes ? kOBytes : kKBytes];
  float (*s_o)[32][D + 1] = reinterpret_cast<float (*)[32][D + 1]>(s_mem);
  __shared__ float s_ml[kWaves][32][2];

  // (tile, split, KV head, sequence, layer), late tiles first
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lrow = lane & 31, half = lane >> 5;
  const int G = a.group;
  const int n_slots = a.n_split_max * (kSolo ? kF32Units : 1);
  const F32Item it = f32_item(a, a.n_qt, n_slots);
  const int tile = a.n_qt - 1 - it.tile, slot = it.slot, g = it.g, b = it.b, l = it.l;   // slot: split, or unit of one
  const int ctx = a.ctx_lens[b];
  if (ctx < 0 || ctx > a.max_ctx_len) return;

  const int pair = tile * 32 + lrow;
  const int lg = 31 - __builtin_clz(G);                        // G is 1, 2, 4 or 8
  const int row = pair >> lg, h = g * G + (pair & (G - 1));
  const bool row_ok = row < a.chunk;
  const int first = tile * 32 >> lg, last = min(tile * 32 + 31 >> lg, a.chunk - 1);
  const int W = layer_window(a, l);
  const int row_n = ctx + row, row_lo = window_start(W, row_n + 1);
  const int mask_lo = window_start(W, ctx + last + 1);        // keys below it are masked for some row
  const int tile_lo = window_start(W, ctx + first + 1);       // the tile's rows see keys in [tile_lo, tile_hi)
  const int tile_hi = ctx + last + 1;
  constexpr int kSlotKeys = kSolo ? kUnitKeys : kSplit, kWaveKeys = kSlotKeys / kWaves;
  if (slot * kSlotKeys >= tile_hi || (slot + 1) * kSlotKeys <= tile_lo) return;
  // this wave's keys, in whole blocks of 32
  const int key_end = min(slot * kSlotKeys + (wave + 1) * kWaveKeys, tile_hi);
  const int key_begin = max(slot * kSlotKeys + wave * kWaveKeys, tile_lo & ~31);
  const int n_blocks = key_end > key_begin ? (key_end - key_begin + 31) / 32 : 0;

  const int64_t lbase = (int64_t)(a.layer0 + l) * a.layer_elems;
  const float* kpool = reinterpret_cast<const float*>(a.k_pool) + lbase;
  const float* vpool = reinterpret_cast<const float*>(a.v_pool) + lbase;
  const int32_t* bt = a.block_tables + (int64_t)b * a.max_pages;
  const int last_page = (tile_hi - 1) / kPage;
  // page ids of the wave's keys (8 pages), one per lane
  const int page0 = key_begin / kPage;
  const int32_t pg = bt[min(page0 + (lane & 15), last_page)];
  auto page_row = [&](int page_slot) -> int64_t {              // first row of the (page, head) slab
    int32_t page = __builtin_amdgcn_readlane(pg, min(page_slot, 15));
    page = (page >= 0 && page < a.n_pages) ? page : 0;
    return ((int64_t)page * a.Hkv + g) * kPage;
  };

  // queries: dims 8 j + 4 half + e; in registers up to head_dim 128, above it in LDS (the K layout)
  FloatVec<4> q[kStaged ? NJ : 1];
  {
    const float* qp = reinterpret_cast<const float*>(a.q) +
                      ((((int64_t)l * a.batch + b) * a.chunk + (row_ok ? row : 0)) * a.Hq + h) * D + 4 * half;
    if constexpr (kStaged) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) q[j] = __builtin_bit_cast(FloatVec<4>, row_ok ? ld16(qp + 8 * j) : make_uint4(0, 0, 0, 0));
    } else {
#pragma unroll
      for (int j = 0; j < NJ / kWaves; ++j) {
        const int jj = wave * (NJ / kWaves) + j;
        st16(s_mem + lrow * RB + 16 * ((2 * jj + half) ^ (lrow & 15)), row_ok ? ld16(qp + 8 * jj) : make_uint4(0, 0, 0, 0));
      }
      __syncthreads();
    }
  }

  f32x16 o[ND];
  float m_run, l_run;

  // K rows of block i: lane % 32's row; V rows of block i: key 8 (r / 4) + 4 half + r % 4.  Rows past the
  // range are rows of a page of the pool: K's are masked, V's are replaced by zeros.
  auto k_ptr = [&](int i) -> const float* {
    const int64_t ra = page_row(2 * i), rb = page_row(2 * i + 1);
    return kpool + ((lrow < kPage ? ra : rb) + lrow % kPage) * D + 4 * half;
  };
  FloatVec<4> kf[LK];
  // Up to head_dim 128 a block's K goes through the wave's own LDS (buffer_load ... lds, 1 KiB of
  // consecutive bytes per load; 16-byte chunks at position chunk ^ (row mod 16)): a lane's 16 bytes of
  // a row straight from L2 took ~90 cycles a load, as long as the MFMAs.  The next block's is
  // requested once this one's has been read, and lands during P V.
  lds_char* const k_lds = (lds_char*)(lds_void*)(s_mem + (kStaged ? wave * 32 * RB : 0));
  constexpr int RPL = 64 / NCH > 0 ? 64 / NCH : 1;
  const int k_r = lane / NCH;
  const uint32_t k_off = k_r * RB + 16 * ((lane % NCH) ^ (k_r & 15));
  const uint32_t k_lane = lrow * RB + 16 * (half ^ (lrow & 15));
  auto stage_k = [&](int i) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int rows = __builtin_amdgcn_readfirstlane(min(max(tile_hi - (key_begin + 32 * i + kPage * p), 0), kPage));
      const int64_t off = __builtin_amdgcn_readfirstlane((int)(page_row(2 * i + p) / kPage)) * (int64_t)kPage * D;
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(kpool + off), 0, rows * RB, kBufferWord3);
#pragma unroll
      for (int j = 0; j < kPage / RPL; ++j) {
        const uint32_t at = j * RPL * RB + (k_off ^ (uint32_t)(16 * ((j * RPL) & 15)));
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(k_lds + (p * kPage + j * RPL) * RB), 16, at, 0, 0, 0);
      }
    }
  };
  auto take_finite = [](FloatVec<NB>& v) {
    FloatVec<NB> rest;
#pragma unroll
    for (int d = 0; d < NB; ++d) {
      const bool ok = fabsf(v.x[d]) <= FLT_MAX;
      rest.x[d] = ok ? 0.0f : v.x[d];
      v.x[d] = ok ? v.x[d] : 0.0f;
    }
    return rest;
  };
  // the values `bad` of keys `key` (lanes 0-31) and key + 4 (lanes 32-63), weighted p, for the rows that see them
  auto add_seen = [&](f32x16 (&ob)[NB], const FloatVec<NB>& bad, float p, int key) {
    bool any = false;
#pragma unroll
    for (int d = 0; d < NB; ++d) any = any || bad.x[d] != 0.0f;
    if (__builtin_amdgcn_ballot_w64(any) == 0) return;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const bool sees = key + 4 * hf <= row_n && key + 4 * hf >= row_lo;
#pragma unroll
      for (int d = 0; d < NB; ++d) {
        const f32x16 t = __builtin_amdgcn_mfma_f32_32x32x2f32(half == hf ? bad.x[d] : 0.0f, p, ob[d], 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) ob[d][r] = sees ? t[r] : ob[d][r];
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // The wave's blocks.  A masked key weighs 0, and 0 times an Inf or NaN among its values would reach the
  // rows that do not see it.  Only if a row's result is not finite are the blocks taken again, `careful`: such
  // values count for the rows that see their key alone.
  for (bool careful = false;; careful = true) {
    const float* kp = k_ptr(0);
    const float* kp_next = kp;
    m_run = -INFINITY;
    l_run = 0.0f;
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[d][r] = 0.0f;
    if (n_blocks > 0) {
      if constexpr (kStaged) {
        stage_k(0);
      } else {
#pragma unroll
        for (int j = 0; j < LK; ++j) kf[j] = __builtin_bit_cast(FloatVec<4>, ld16(kp + 8 * j));
      }
    }
    for (int i = 0; i < n_blocks; ++i) {
      const int kb = key_begin + 32 * i;
      kp_next = k_ptr(i + 1);                                    // past the last block: rows never used
      const int64_t va = page_row(2 * i), vb = page_row(2 * i + 1);
      const float* vp0 = vpool + (va + 4 * half) * D + ND * lrow;
      const float* vp1 = vpool + (vb + 4 * half) * D + ND * lrow;
      FloatVec<NB> vf[LV];
      auto vfetch = [&](int x) {                                 // step x mod 16 of pass x / 16
        const int r = x % 16;
        const float* p = (r < 8 ? vp0 : vp1) + (8 * ((r / 4) & 1) + r % 4) * D + NB * (x / 16);
        vf[x % LV] = *reinterpret_cast<const FloatVec<NB>*>(p);
      };

      f32x16 c[4];
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int r = 0; r < 16; ++r) c[x][r] = 0.0f;
      auto kread = [&](int j) -> FloatVec<4> {
        return __builtin_bit_cast(FloatVec<4>, *reinterpret_cast<const lds_u32x4*>(k_lds + (k_lane ^ (uint32_t)(32 * j))));
      };
      if constexpr (kStaged) {
        __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0): the block's K
        asm volatile("" ::: "memory");
#pragma unroll
        for (int j = 0; j < 4; ++j) kf[j] = kread(j);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const FloatVec<4> k = kf[j % LK];
        if constexpr (kStaged) {
          if (j + 4 < NJ) kf[(j + 4) % LK] = kread(j + 4);
        } else {
          kf[j % LK] = __builtin_bit_cast(FloatVec<4>, ld16((j + LK < NJ ? kp : kp_next) + 8 * ((j + LK) % NJ)));
        }
        if (j >= NJ - LV) vfetch(j - (NJ - LV));
        const FloatVec<4> qj = kStaged ? q[kStaged ? j : 0] : kread(j);
#pragma unroll
        for (int e = 0; e < 4; ++e) c[j % 4] = __builtin_amdgcn_mfma_f32_32x32x2f32(k.x[e], qj.x[e], c[j % 4], 0, 0, 0);
      }
      kp = kp_next;
      if constexpr (kStaged) {
        __builtin_amdgcn_s_waitcnt(0xC07F);                      // lgkmcnt(0): the reads have returned
        asm volatile("" ::: "memory");
        if (i + 1 < n_blocks) stage_k(i + 1);
      }
      f32x16 s;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = (c[0][r] + c[1][r]) + (c[2][r] + c[3][r]);
      if (kb + 31 > ctx + first || kb < mask_lo) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = kb + half * 4 + (r >> 2) * 8 + (r & 3);
          s[r] = (key <= row_n && key >= row_lo) ? s[r] : -INFINITY;
        }
      }
      float mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[r]);
      const float2 mh = halves32(mx);
      // the block's own state (reference: its largest score), folded into the wave's
      const float m_blk = fmaxf(mh.x, mh.y) * a.scale_log2;
      const float m_ref = m_blk == -INFINITY ? 0.0f : m_blk;     // no key seen: every p is 0
      float psum = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[r] = block_weight(s[r], a.scale_log2, m_ref);
        psum += s[r];
      }
      const float2 ph = halves32(psum);
      const float m_new = fmaxf(m_run, m_blk);
      const float f_run = merge_factor(m_run, m_new), f_blk = merge_factor(m_blk, m_new);
      l_run = fold(l_run, f_run, ph.x + ph.y, f_blk);
      m_run = m_new;
      const bool edge = kb + 32 > tile_hi || kb < tile_lo;
#pragma unroll
      for (int pass = 0; pass < ND / NB; ++pass) {
        f32x16 ob[NB];
#pragma unroll
        for (int d = 0; d < NB; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) ob[d][r] = 0.0f;
        auto pv = [&](auto masked) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int x = 16 * pass + r;
            FloatVec<NB> v = vf[x % LV];
            if (x + LV < 16 * (ND / NB)) vfetch(x + LV);
            FloatVec<NB> bad;                                    // its Inf and NaN values, zeros elsewhere
            if constexpr (decltype(masked)::value) {
              const int key = kb + half * 4 + (r >> 2) * 8 + (r & 3);
              const bool in = key >= tile_lo && key < tile_hi;
#pragma unroll
              for (int d = 0; d < NB; ++d) v.x[d] = in ? v.x[d] : 0.0f;
              if (careful) bad = take_finite(v);
            }
#pragma unroll
            for (int d = 0; d < NB; ++d) ob[d] = __builtin_amdgcn_mfma_f32_32x32x2f32(v.x[d], s[r], ob[d], 0, 0, 0);
            if constexpr (decltype(masked)::value) {
              if (careful) add_seen(ob, bad, s[r], kb + (r >> 2) * 8 + (r & 3));
            }
          }
        };
        if (edge || careful)
          pv(std::true_type{});
        else
          pv(std::false_type{});
#pragma unroll
        for (int d = 0; d < NB; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[NB * pass + d][r] = fold(o[NB * pass + d][r], f_run, ob[d][r], f_blk);
      }
    }
    if (careful || __builtin_amdgcn_ballot_w64(row_ok && !all_finite(o)) == 0) break;
  }

  __syncthreads();                                             // every wave is past its K blocks
  // ---- the four waves' states in order: O^T element r of block d is dim ND (8 (r / 4) + 4 half + r % 4) + d
  // of pair lrow
#pragma unroll
  for (int d = 0; d < ND; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) s_o[wave][lrow][ND * (8 * (r >> 2) + 4 * half + (r & 3)) + d] = o[d][r];
  if (half == 0) {
    s_ml[wave][lrow][0] = m_run;
    s_ml[wave][lrow][1] = l_run;
  }
  __syncthreads();
  for (int t = threadIdx.x; t < 32 * D; t += 64 * kWaves) {
    const int p = t / D, d = t % D;
    const int prow = tile * 32 + p >> lg, ph = g * G + (tile * 32 + p & (G - 1));
    if (prow >= a.chunk) break;
    float m = -INFINITY, lsum = 0.0f, v = 0.0f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) fold_state(m, lsum, v, s_ml[w][p][0], s_ml[w][p][1], s_o[w][p][d]);
    const int64_t rh = (((int64_t)l * a.batch + b) * a.chunk + prow) * a.Hq + ph;
    if (a.part_acc == nullptr) {
      a.out[rh * D + d] = v / lsum;
    } else {
      const int64_t pidx = rh * n_slots + slot;
      a.part_acc[pidx * D + d] = v;
      if (d == 0) *reinterpret_cast<float2*>(a.part_ml + pidx * 2) = make_float2(m, lsum);
    }
  }
}

// Small calls: P pairs at a time on the vector ALUs, with the operations of a 32-pair tile in its order (the matrix
// cores' step is an fma chain, lanes 0-31's product first), so with its bytes.  Workgroup = (layer, sequence,
// KV head, tile of P pairs, unit of 128 keys), two waves of 64 keys: a key per lane for the scores, then the weights
// through LDS and D / 64 dimensions a lane for the values.  A tile's 32 pairs are mostly padding in such calls, its
// waves run their blocks one after the other, and its code (20 to 77 KB) takes longer to arrive than the work: what
// bounds this one is the round trips (page, K and V rows requested together, the rest of K) and its 10 to 14 KB.
// Queries as scalar loads, a miss each, cost 5 us more at head_dim 256; eight pairs a workgroup, 40 KB of code, 20.
template <int D, int P>
__global__ __launch_bounds__(128) void prefill_f32_narrow_kernel(const PrefillArgs a) {
  constexpr int E = D / 64;                                    // dimensions per lane
  constexpr int LK = 8;                                        // K loads ahead, 8 dimensions each
  __shared__ __attribute__((aligned(16))) float s_q[P][D];
  __shared__ __attribute__((aligned(16))) float s_p[2][P][64];
  __shared__ float s_o[2][P][D];                               // wave 1's blocks
  __shared__ float2 s_ml[2][P];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int G = a.group, lg = 31 - __builtin_clz(G);
  const int n_nt = narrow_tiles(a, P);
  const int n_slots = a.n_split_max * kF32Units;
  const F32Item it = f32_item(a, n_nt, n_slots);
  const int tile = it.tile, slot = it.slot, g = it.g, b = it.b, l = it.l;
  const int ctx = a.ctx_lens[b];
  if (ctx < 0 || ctx > a.max_ctx_len) return;
  const int W = layer_window(a, l);
  const int first = tile * P >> lg, last = min(tile * P + P - 1 >> lg, a.chunk - 1);
  const int tile_lo = window_start(W, ctx + first + 1), tile_hi = ctx + last + 1;
  if (slot * kUnitKeys >= tile_hi || (slot + 1) * kUnitKeys <= tile_lo) return;
  const int mask_lo = window_start(W, ctx + last + 1);         // keys below it are masked for some row

  const int64_t lbase = (int64_t)(a.layer0 + l) * a.layer_elems;
  const float* kpool = reinterpret_cast<const float*>(a.k_pool) + lbase;
  const float* vpool = reinterpret_cast<const float*>(a.v_pool) + lbase;
  const int key0 = slot * kUnitKeys + 64 * wave;               // lane's key: key0 + lane
  const int key = key0 + lane;
  int32_t page = a.block_tables[(int64_t)b * a.max_pages + min(key, tile_hi - 1) / kPage];
  page = (page >= 0 && page < a.n_pages) ? page : 0;
  const int64_t slab = ((int64_t)page * a.Hkv + g) * kPage;    // the lane's key's (page, head)

  // pair p's row and query (a pair past the chunk takes the last row's and is not written)
  auto row_of = [&](int p) { return min(tile * P + p >> lg, a.chunk - 1); };
  auto head_row = [&](int p) -> int64_t {
    return (((int64_t)l * a.batch + b) * a.chunk + row_of(p)) * a.Hq + g * G + (tile * P + p & (G - 1));
  };
  // V rows of a block, requested before its weights are known.  Rows past tile_hi are rows of a page of the pool
  // that no pair sees.
  FloatVec<E> v[32];
  auto vfetch = [&](int blk) {
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int64_t pg = __builtin_amdgcn_readlane(page, 32 * blk + kPage * x);
      const float* vr = vpool + (pg * a.Hkv + g) * kPage * D + E * lane;
#pragma unroll
      for (int k = 0; k < kPage; ++k) v[kPage * x + k] = *reinterpret_cast<const FloatVec<E>*>(vr + k * D);
    }
  };
  float m_blk[P], w[P];
  const bool any_key = key0 < tile_hi && key0 + 64 > tile_lo;
  // the queries, 16 bytes a thread; the K and V rows are requested before they are waited for
  constexpr int NQ = P * D / 4;
  uint4 q_raw = make_uint4(0, 0, 0, 0);
  static_assert(NQ <= 128, "a chunk of the queries per thread");
  if ((int)threadIdx.x < NQ) {
    int64_t qr = 0;
#pragma unroll
    for (int p = 0; p < P; ++p) qr = (int)threadIdx.x / (D / 4) == p ? head_row(p) : qr;
    q_raw = ld16(reinterpret_cast<const float*>(a.q) + qr * D + 4 * (threadIdx.x % (D / 4)));
  }
  FloatVec<8> kf[LK];
  const float* kr = kpool + (slab + lane % kPage) * D;
  if (any_key) {
#pragma unroll
    for (int j = 0; j < LK; ++j) kf[j] = load8(kr + 8 * j);
    vfetch(0);
  }
  if ((int)threadIdx.x < NQ) st16(&s_q[0][0] + 4 * threadIdx.x, q_raw);
  __syncthreads();
  if (any_key) {
    float c[P][4];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int x = 0; x < 4; ++x) c[p][x] = 0.0f;
#pragma unroll 1
    for (int j0 = 0; j0 < D / 8; j0 += LK) {
#pragma unroll
      for (int x = 0; x < LK; ++x) {
        const FloatVec<8> k = kf[x];
        kf[x] = load8(kr + 8 * min(j0 + x + LK, D / 8 - 1));
#pragma unroll
        for (int p = 0; p < P; ++p) {
          const FloatVec<8> q = load8(&s_q[p][8 * (j0 + x)]);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            c[p][x % 4] = fmaf(k.x[e], q.x[e], c[p][x % 4]);
            c[p][x % 4] = fmaf(k.x[e + 4], q.x[e + 4], c[p][x % 4]);
          }
        }
      }
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int row_n = ctx + row_of(p);
      const float s = (c[p][0] + c[p][1]) + (c[p][2] + c[p][3]);
      w[p] = key <= row_n && key >= window_start(W, row_n + 1) ? s : -INFINITY;
      float mx = w[p];
#pragma unroll
      for (int x = 16; x >= 1; x >>= 1) mx = fmaxf(mx, __shfl_xor(mx, x));
      m_blk[p] = mx * a.scale_log2;                            // of the lane's half: its block's
      const float m_ref = m_blk[p] == -INFINITY ? 0.0f : m_blk[p];
      s_p[wave][p][lane] = block_weight(w[p], a.scale_log2, m_ref);
    }
  } else {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      m_blk[p] = -INFINITY;
      s_p[wave][p][lane] = 0.0f;
    }
  }
  __syncthreads();

  // the wave's two blocks: (reference, sum, O) each
  float m[P], lsum[P], o[P][E];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    m[p] = -INFINITY;
    lsum[p] = 0.0f;
#pragma unroll
    for (int e = 0; e < E; ++e) o[p][e] = 0.0f;
  }
#pragma unroll 1
  for (int blk = 0; blk < 2; ++blk) {
    const int kb = key0 + 32 * blk;
    float ps[P][2], ob[P][E];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      ps[p][0] = ps[p][1] = 0.0f;
#pragma unroll
      for (int e = 0; e < E; ++e) ob[p][e] = 0.0f;
    }
    // a key that a pair does not see adds 0 times 0, whatever its values are
    const bool masked = kb + 31 > ctx + first || kb < mask_lo;
    auto octet = [&](int k8) {
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const float4 wa = *reinterpret_cast<const float4*>(&s_p[wave][p][32 * blk + k8]);
        const float4 wb = *reinterpret_cast<const float4*>(&s_p[wave][p][32 * blk + k8 + 4]);
        const float wt[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
        const int row_n = ctx + row_of(p), row_lo = window_start(W, row_n + 1);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            const int x = t + 4 * hf, kk = kb + k8 + x;
            const bool sees = !masked || (kk <= row_n && kk >= row_lo);
            ps[p][hf] += wt[x];
#pragma unroll
            for (int e = 0; e < E; ++e) ob[p][e] = fmaf(sees ? v[k8 + x].x[e] : 0.0f, wt[x], ob[p][e]);
          }
      }
    };
    if (kb < tile_hi && kb + 32 > tile_lo) {
#pragma unroll
      for (int k8 = 0; k8 < 32; k8 += 8) octet(k8);
    }
    if (blk == 0) vfetch(1);
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const float mb = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(m_blk[p]), 32 * blk));
      const float lb = ps[p][0] + ps[p][1];
      if (wave == 0) {
        const float m_new = fmaxf(m[p], mb), f = merge_factor(m[p], m_new), fb = merge_factor(mb, m_new);
        lsum[p] = fold(lsum[p], f, lb, fb);
#pragma unroll
        for (int e = 0; e < E; ++e) o[p][e] = fold(o[p][e], f, ob[p][e], fb);
        m[p] = m_new;
      } else {
#pragma unroll
        for (int e = 0; e < E; ++e) s_o[blk][p][E * lane + e] = ob[p][e];
        if (lane == 0) s_ml[blk][p] = make_float2(mb, lb);
      }
    }
  }
  __syncthreads();
  if (wave == 1) return;
#pragma unroll
  for (int p = 0; p < P; ++p) {
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      const float2 ml = s_ml[blk][p];
      const float m_new = fmaxf(m[p], ml.x), f = merge_factor(m[p], m_new), fb = merge_factor(ml.x, m_new);
      lsum[p] = fold(lsum[p], f, ml.y, fb);
#pragma unroll
      for (int e = 0; e < E; ++e) o[p][e] = fold(o[p][e], f, s_o[blk][p][E * lane + e], fb);
      m[p] = m_new;
    }
    if (tile * P + p >= a.chunk * G) break;
    const int64_t rh = head_row(p);
    FloatVec<E> out;
    if (a.part_acc == nullptr) {
#pragma unroll
      for (int e = 0; e < E; ++e) out.x[e] = o[p][e] / lsum[p];
      *reinterpret_cast<FloatVec<E>*>(a.out + rh * D + E * lane) = out;
    } else {
      const int64_t pidx = rh * n_slots + slot;
#pragma unroll
      for (int e = 0; e < E; ++e) out.x[e] = o[p][e];
      *reinterpret_cast<FloatVec<E>*>(a.part_acc + pidx * D + E * lane) = out;
      if (lane == 0) *reinterpret_cast<float2*>(a.part_ml + pidx * 2) = make_float2(m[p], lsum[p]);
    }
  }
}

// The units' partials of a row in the order the one-workgroup split takes them, then the splits as
// combine_splits does.  One element per lane.
// NS: splits whose loads are in flight.
template <int NS>
__global__ __launch_bounds__(256) void prefill_f32_units_kernel(const PrefillArgs a, uint32_t n) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const uint32_t D = a.D, row_head = i / D;
  uint32_t id = row_head / (uint32_t)a.Hq;
  const int row = (int)(id % (uint32_t)a.chunk);
  id /= (uint32_t)a.chunk;
  const int b = (int)(id % (uint32_t)a.batch), l = (int)(id / (uint32_t)a.batch);
  const int ctx = a.ctx_lens[b];
  if (ctx < 0 || ctx > a.max_ctx_len) return;
  const int n_keys = ctx + row + 1;
  const int u0 = window_start(layer_window(a, l), n_keys) / kUnitKeys, u1 = (n_keys - 1) / kUnitKeys;
  const int64_t p0 = (int64_t)row_head * a.n_split_max * kF32Units;
  const float2* ml = reinterpret_cast<const float2*>(a.part_ml) + p0;
  const float* acc = a.part_acc + p0 * D + i % D;
  constexpr int U = NS * kF32Units, M = 2 * U;                 // units whose loads are in flight
  float m = -INFINITY;
  for (int u = u0; u <= u1; u += M) {
    float mv[M];
#pragma unroll
    for (int x = 0; x < M; ++x) mv[x] = ml[min(u + x, u1)].x;
#pragma unroll
    for (int x = 0; x < M; ++x) m = fmaxf(m, mv[x]);
  }
  float lsum = 0.0f, o = 0.0f;
  for (int s = u0 / kF32Units; s <= u1 / kF32Units; s += NS) {
    float2 pv[U];
    float av[U];
#pragma unroll
    for (int x = 0; x < U; ++x) {
      const int u = min(max(s * kF32Units + x, u0), u1);
      pv[x] = ml[u];
      av[x] = acc[(int64_t)u * a.D];
    }
#pragma unroll
    for (int y = 0; y < NS; ++y) {
      float sm = -INFINITY, sl = 0.0f, sv = 0.0f;
#pragma unroll
      for (int w = 0; w < kF32Units; ++w) {
        const int x = y * kF32Units + w, u = s * kF32Units + x;
        if (u >= u0 && u <= u1) fold_state(sm, sl, sv, pv[x].x, pv[x].y, av[x]);
      }
      const float f = merge_factor(sm, m);
      lsum = fmaf(sl, f, lsum);
      o = fmaf(sv, f, o);
    }
  }
  a.out[i] = o / lsum;
}

hipError_t launch_narrow(const PrefillArgs& a, hipStream_t stream) {
  constexpr int P = 2;
  const int64_t n_wg = (int64_t)a.n_layers * a.batch * a.Hkv * a.n_split_max * kF32Units * narrow_tiles(a, P);
  const dim3 grid((unsigned)n_wg);
  switch (a.D) {
    case 64: prefill_f32_narrow_kernel<64, P><<<grid, 128, 0, stream>>>(a); break;
    case 128: prefill_f32_narrow_kernel<128, P><<<grid, 128, 0, stream>>>(a); break;
    case 256: prefill_f32_narrow_kernel<256, P><<<grid, 128, 0, stream>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <bool kSolo>
hipError_t launch(const PrefillArgs& a, hipStream_t stream) {
  const dim3 grid((unsigned)(prefill_f32_workgroups(a) * (kSolo ? kF32Units : 1)));
  switch (a.D) {
    case 64: prefill_f32_kernel<64, kSolo><<<grid, 64 * kWaves, 0, stream>>>(a); break;
    case 128: prefill_f32_kernel<128, kSolo><<<grid, 64 * kWaves, 0, stream>>>(a); break;
    case 256: prefill_f32_kernel<256, kSolo><<<grid, 64 * kWaves, 0, stream>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_prefill_f32(const PrefillArgs& a, F32Form form, hipStream_t stream) {
  const hipError_t e = form == F32Form::kNarrow ? launch_narrow(a, stream)
                       : form == F32Form::kUnits ? launch<true>(a, stream)
                                                 : launch<false>(a, stream);
  if (e != hipSuccess || a.part_acc == nullptr) return e;
  if (form == F32Form::kSplits) return launch_prefill_segments(a, stream);
  const int64_t n = (int64_t)a.n_layers * a.batch * a.chunk * a.Hq * a.D;   // few workgroups: below 2^31
  const dim3 grid((unsigned)((n + 255) / 256));
  // one row over 8k keys 26 -> 24 us with four splits at a time; over 1k keys 15.6 with two, 16.5 with four, for the
  // code is longer
  if (a.n_split_max <= 4)
    prefill_f32_units_kernel<2><<<grid, 256, 0, stream>>>(a, (uint32_t)n);
  else
    prefill_f32_units_kernel<4><<<grid, 256, 0, stream>>>(a, (uint32_t)n);
  return hipGetLastError();
}

}  // namespace kvg
