// Decode attention of bf16 and fp8 caches on MFMA: one new token per sequence, split over keys.
//
// Work item = (layer, sequence, KV head g, split s of kSplit = 512 keys), one wave each.  The
// split is four units of 128 keys (a window's last one up to 15 keys longer: split_base); each unit
// starts from an empty softmax state, and the units of a split are merged in order.  Splits are
// combined in ascending order by the merge kernels.  Everything is a function of the row's own length
// and window, so a sequence's bytes depend neither on its batch nor on the pages' places.
//
// What bounds it: HBM, when the launch fills the chip.  Keys and values go from the pages straight
// into LDS (buffer_load ... lds, whole (page, head) slabs, 1 KiB of consecutive bytes per
// instruction), kStages stages deep, without a register; a workgroup is one wave, so a CU holds
// three to ten (launch_decode_type) and their starts and ends overlap.  The arithmetic is
// small beside that: a 16-key tile's scores for up to 8 query heads are D / 32
// v_mfma_f32_16x16x32_bf16 (A = 16 keys, B = the heads' queries: bf16 high parts in columns 0-7, low
// parts in columns 8-15, the two halves added by one row rotation), the weights leave the
// accumulator in the order the next operand needs (high parts in columns 0-7, remainders in columns
// 8-15, so a weight keeps 16 significant bits at no cost), and O^T += V^T P^T takes one MFMA per
// 16 dimensions with V read transposed from LDS (ds_read_b64_tr).  On the vector ALUs (16-lane teams,
// one dot product per key and head) a pair of keys took ~200 instructions in a row, which bound
// every launch that left CUs idle.  A wave alone is slower than a workgroup of those was (20 us for 512
// keys of 512-byte rows), so a launch's last round weighs more here: 1,728 splits 152 us against 147 there.
//
// kSolo: a wave per unit instead of per split, for launches that leave CUs idle; the four units of a
// split leave four partials, which merge_splits_kernel merges with the same operations in the
// same order, so the bytes are the same.
#include "kvg_launch.h"
#include "kvg_mfma.h"
#include "kvg_rows.h"

#include <math.h>

#include <type_traits>

namespace kvg {

namespace {

constexpr int kFewKeys = 64;           // rows of at most so many keys take exact weights
constexpr int kStream = 2;             // buffer load policy: nontemporal (every row is read once)
constexpr int kLgkmWait = 0xC07F;      // s_waitcnt operand: lgkmcnt(0) alone
// s_waitcnt operand that waits for vmcnt <= n alone (gfx9 encoding: bits 3:0 and 15:14)
constexpr int vm_wait(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

// x of lanes with an even and with an odd index / 16, to both (as halves32 for index / 32)
__device__ __forceinline__ float2 rows16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return make_float2(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max_over_groups(float x) {
  const float2 a = rows16(x);
  const float2 b = halves32(fmaxf(a.x, a.y));
  return fmaxf(b.x, b.y);
}
__device__ __forceinline__ float sum_over_groups(float x) {
  const float2 a = rows16(x);
  const float2 b = halves32(a.x + a.y);
  return b.x + b.y;
}
// x + the value eight lanes on in the same 16-lane row
__device__ __forceinline__ float add_ror8(float x) {
  return x + __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(x), 0x128, 0xF, 0xF, true));
}

// LDS rows hold their 16-byte chunks at position chunk ^ swizzle(row).  Rows of RB bytes: 256 / RB
// of them share a 256-byte line of the banks.
//   K: 16 rows x one chunk per 16 (fp8: 32) lanes; V: bf16 eight rows x two chunks, fp8 rows
//   {0..7, 16..23} (+ 8) x one chunk.  Both are XOR-linear in the row bits.
template <int RB, bool kFp8>
struct SwzDecode {
  __device__ static __forceinline__ int k(int r) {
    return RB >= 256 ? (r & 15) : RB == 128 ? ((r >> 1) & 7) : ((r >> 2) & 3);
  }
  __device__ static __forceinline__ int v(int r) {
    if constexpr (!kFp8) return RB >= 256 ? 2 * (r & 7) : 2 * ((r >> 1) & 3);
    return RB == 256   ? (r & 7) | (((r >> 4) & 1) << 3)
           : RB == 128 ? ((r >> 1) & 3) | (((r >> 4) & 1) << 2)
                       : ((r >> 2) & 1) | (((r >> 4) & 1) << 1);
  }
};

typedef short i16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// A workgroup is one wave: its LDS writes are visible to it, and its reads done, once lgkmcnt is 0.
__device__ __forceinline__ void lds_ready() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(kLgkmWait);
  asm volatile("" ::: "memory");
}

template <int S, int BYTES>
__device__ __forceinline__ uint4* stage_memory() {
  __shared__ __attribute__((aligned(1024))) uint4 mem[BYTES / 16];
  return mem;
}

// kStages: stages of K and V in flight, per wave
template <typename T, int D, bool kSolo, int kStages>
__global__ __launch_bounds__(64, kSolo ? 1 : 2) void decode_mfma_kernel(const DecodeArgs a) {
  constexpr bool kFp8 = sizeof(T) == 1;
  using R = uint16_t;                                // raw inputs are bf16
  constexpr int RB = D * (int)sizeof(T);             // bytes per cache row
  constexpr int NCH = RB / 16;
  constexpr int kStageBytes = decode_stage_bytes(RB);     // K and V of one stage
  constexpr int SK = kStageBytes / 2 / RB;           // keys per stage
  constexpr int PS = SK / kPage;                     // pages per stage
  constexpr int BK = SK < 32 ? SK : 32;              // keys per softmax block
  constexpr int NTL = BK / 16;                       // 16-key tiles of a block
  constexpr int NS = D / 32;                         // MFMA steps of a score tile
  constexpr int ND = D / 16;                         // 16-wide blocks of head_dim
  constexpr int kLoads = kStageBytes / 1024;         // direct loads per stage
  constexpr int kUnitStages = kUnit / SK;
  static_assert(kUnit % SK == 0 && SK % BK == 0 && (kStages - 1) * kLoads <= 63, "stage");
  using SW = SwzDecode<RB, kFp8>;
  // one LDS object per stage, so that the compiler can tell the stage being read from those
  // being loaded; K rows, then V rows
  auto stage_mem = [&](auto st) -> uint4* { return stage_memory<decltype(st)::value, kStageBytes>(); };

  // ---- work item (the order of the fp32 decode: sequence fastest; with a shared window runs of 64
  // items go to one XCD)
  int64_t w = blockIdx.x;
  int unit0 = 0;
  if constexpr (kSolo) {
    unit0 = (int)(w & 3);
    w >>= 2;
  }
  if (a.shared_order) {
    constexpr int64_t CH = 64;
    const int64_t full = (int64_t)gridDim.x / (kSolo ? 4 : 1) / (8 * CH) * (8 * CH);
    if (w < full) {
      const int64_t g8 = w / 8;
      w = ((g8 / CH) * 8 + w % 8) * CH + g8 % CH;
    }
  }
  const DecodeItem item = decode_item(a, w);
  const int b = item.b, si = item.si, g = item.g, l = item.l;
  const int lane = threadIdx.x;
  const int G = a.group;
  const int64_t tok = (int64_t)l * a.batch + b;
  const int32_t* bt = a.block_tables + (int64_t)b * a.max_pages;
  const int win = layer_window(a, l);
  const int s = (win == 0 ? a.n_shared_split : 0) + si;


  // ---- requested before the context length is known, which they do not depend on: the raw rows
  // of this lane's query chunks and of the new token's, its frequencies, and (without a window) the
  // page ids.  The stages' loads queue behind them, so nothing waits for a stage to get them.
  const int64_t head0 = tok * a.Hq + (int64_t)g * G;
  const int col = lane & 15, grp = lane >> 4;
  const int head = col & 7;
  const R* qrow = reinterpret_cast<const R*>(a.q_raw) + head0 * D;
  const int pair_x = a.pairing == 0 ? D / 16 : 0;    // half pairing: a chunk's partner is D / 2 away
  constexpr int NCHR = D / 8;                        // 16-byte chunks of a raw row
  constexpr int QC = 8 * NCHR / 64;                  // query chunks per lane, 8 heads
  uint4 qa[QC], qb[QC];
#pragma unroll
  for (int i = 0; i < QC; ++i) {
    const int c = min(64 * i + lane, G * NCHR - 1);  // chunk c % NCHR of head c / NCHR
    qa[i] = ld16(qrow + c * 8);
    qb[i] = ld16(qrow + (c ^ pair_x) * 8);
  }
  constexpr int P = Elem<T>::kPerVec / 8;            // raw chunks per storage chunk
  const R* kraw = reinterpret_cast<const R*>(a.k_raw) + (tok * a.Hkv + g) * D;
  const R* vraw = reinterpret_cast<const R*>(a.v_raw) + (tok * a.Hkv + g) * D;
  const int nc = min(lane, NCH - 1);
  uint4 ka[P], kb[P], va[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    ka[p] = ld16(kraw + (nc * P + p) * 8);
    kb[p] = ld16(kraw + ((nc * P + p) ^ pair_x) * 8);
    va[p] = ld16(vraw + (nc * P + p) * 8);
  }
  constexpr int NTH = (D / 2 + 63) / 64;
  double theta[NTH];
#pragma unroll
  for (int i = 0; i < NTH; ++i) theta[i] = a.theta[min(lane + 64 * i, D / 2 - 1)];
  int32_t pg = bt[min((s * kSplit + unit0 * kUnit) / kPage + lane, a.max_pages - 1)];
  __builtin_amdgcn_sched_barrier(0);

  const int ctx = a.ctx_lens[b];
  const int64_t pos = a.start_pos[b] + ctx;
  if (ctx < 0 || ctx > a.max_ctx_len) return;
  const int n_keys = ctx + 1;                        // the new token is key ctx
  const int lo = window_start(win, n_keys);
  const int base = split_base(lo);
  const int n_split = split_count(n_keys, lo);
  if (s >= n_split) return;
  const int k0 = base + s * kSplit + unit0 * kUnit;  // this wave's keys [k0, k1), page aligned
  const bool to_end = s == n_split - 1 && (!kSolo || unit0 == 3);   // the last unit takes what is left
  const int k1 = to_end ? n_keys : min(kSolo ? k0 + kUnit : k0 + kSplit, n_keys);
  if (kSolo && k0 >= k1) return;                     // an empty unit (never read)
  const int n_stages = (k1 - k0 + SK - 1) / SK;
  if (win != 0) pg = bt[min(k0 / kPage + lane, a.max_pages - 1)];   // a split is at most 33 pages
  const bool has_new = ctx < k1;                     // this wave owns the new token

  const int64_t lbase = (int64_t)(a.layer0 + l) * a.layer_elems;
  T* kpool = reinterpret_cast<T*>(a.k_pool) + lbase;
  T* vpool = reinterpret_cast<T*>(a.v_pool) + lbase;
  auto page_of = [&](int p) -> int32_t { return __builtin_amdgcn_readfirstlane(__builtin_amdgcn_readlane(pg, p)); };

  // ---- direct loads of stage i: load j covers slots [64 j, 64 j + 64) of the K rows (then of the V
  // rows): row (64 j + lane) / NCH, position (64 j + lane) % NCH.  A slab's resource ends at its
  // last row below k1, so rows past it read as zeros (weighted 0); past the last stage
  // every resource is empty.  The first stage's value rows below the window are zeros too (an offset
  // past the slab): an Inf or NaN there, times 0, would reach the result.
  constexpr int RPL = 64 / NCH;                      // rows per load
  const int lr = lane / NCH;
  const uint32_t k_off = lr * RB + 16 * ((lane % NCH) ^ SW::k(lr));
  const uint32_t v_off = lr * RB + 16 * ((lane % NCH) ^ SW::v(lr));
  auto issue = [&](auto st, int i, auto first) {
    lds_char* dst = (lds_char*)(lds_void*)stage_mem(st);
#pragma unroll
    for (int p = 0; p < PS; ++p) {
      const int slot = i * PS + p;
      int32_t page = page_of(min(slot, 63));
      page = (page >= 0 && page < a.n_pages) ? page : 0;
      const int rows = __builtin_amdgcn_readfirstlane(min(max(k1 - k0 - slot * kPage, 0), kPage));
      const int64_t off = ((int64_t)page * a.Hkv + g) * kPage * D;
      const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(kpool + off, 0, rows * RB, kBufferWord3);
      const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(vpool + off, 0, rows * RB, kBufferWord3);
#pragma unroll
      for (int j = 0; j < kPage / RPL; ++j) {
        const int r0 = j * RPL;                      // row in the page
        const int rs = p * kPage + r0;               // row in the stage
        const uint32_t ok = r0 * RB + (k_off ^ (16 * SW::k(rs)));
        uint32_t ov = r0 * RB + (v_off ^ (16 * SW::v(rs)));
        if (decltype(first)::value && p == 0) ov = k0 + r0 + lr < lo ? kPage * RB : ov;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (lds_void*)(dst + rs * RB), 16, ok, 0, 0, kStream);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (lds_void*)(dst + SK * RB + rs * RB), 16, ov, 0, 0, kStream);
      }
    }
  };
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  using S2 = std::integral_constant<int, 2>;
  issue(S0{}, 0, std::true_type{});
  if constexpr (kStages > 2) issue(S1{}, 1, std::false_type{});

  // ---- rotation table in the last stage's memory (its first loads come after it is read),
  // rotated queries, the new token's rows (written to the cache, kept for LDS)
  float* cs = reinterpret_cast<float*>(stage_memory<kStages - 1, kStageBytes>());
#pragma unroll
  for (int i = 0; i < NTH; ++i) {
    const int p = lane + 64 * i;
    double sn, cn;
    sincos((double)pos * theta[i], &sn, &cn);
    if (p < D / 2) *reinterpret_cast<float2*>(cs + 2 * p) = make_float2((float)cn, (float)sn);
  }
  lds_ready();
  // the rotated queries as hi and lo parts, [2][G heads][D] bf16 behind the table
  uint4* s_q = reinterpret_cast<uint4*>(cs + D);
#pragma unroll
  for (int i = 0; i < QC; ++i) {
    const int t = 64 * i + lane, c = t % NCHR;
    if (64 * i < G * NCHR) {
      float x[8];
      if (a.pairing == 0) {
        const bool first = c < D / 16;
        rotate_chunk<R>(qa[i], qb[i], first, (first ? c : c - D / 16) * 8, 0, cs, x);
      } else {
        rotate_chunk<R>(qa[i], qa[i], true, c * 4, 1, cs, x);
      }
      uint4 hi, lw;
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const bf16x2 h = __builtin_convertvector((f32x2){x[e], x[e + 1]}, bf16x2);
        (&hi.x)[e / 2] = __builtin_bit_cast(uint32_t, h);
        (&lw.x)[e / 2] = pack_bf16_rne(x[e] - (float)h.x, x[e + 1] - (float)h.y);
      }
      if (t < G * NCHR) {
        s_q[t] = hi;
        s_q[G * NCHR + t] = lw;
      }
    }
  }
  uint4 new_k = make_uint4(0, 0, 0, 0), new_v = new_k;
  if (has_new) {
    float xk[8 * P], xv[8 * P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int c = nc * P + p;
      if (a.pairing == 0) {
        const bool first = c < D / 16;
        rotate_chunk<R>(ka[p], kb[p], first, (first ? c : c - D / 16) * 8, 0, cs, xk + 8 * p);
      } else {
        rotate_chunk<R>(ka[p], ka[p], true, c * 4, 1, cs, xk + 8 * p);
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) xv[8 * p + e] = Elem<R>::get(va[p], e);
    }
    uint32_t wk[4], wv[4];
    pack_words<T, 8 * P>(xk, wk);
    pack_words<T, 8 * P>(xv, wv);
    new_k = make_uint4(wk[0], wk[1], wk[2], wk[3]);
    new_v = make_uint4(wv[0], wv[1], wv[2], wv[3]);
    const int32_t page = page_of((ctx - k0) / kPage);
    if (lane < NCH && page >= 0 && page < a.n_pages) {
      const int64_t roff = (((int64_t)page * a.Hkv + g) * kPage + (ctx % kPage)) * D;
      st16(reinterpret_cast<uint4*>(kpool + roff) + lane, new_k);
      st16(reinterpret_cast<uint4*>(vpool + roff) + lane, new_v);
    }
  }
  lds_ready();
  uint4 q[NS];                                       // B operand: columns 0-7 hi, 8-15 lo, 0 past the heads
  const uint32_t head_mask = head < G ? 0xFFFFFFFFu : 0u;
#pragma unroll
  for (int ss = 0; ss < NS; ++ss) {
    const uint4 v = s_q[((col >> 3) * G + min(head, G - 1)) * NCHR + 4 * ss + grp];
    q[ss] = make_uint4(v.x & head_mask, v.y & head_mask, v.z & head_mask, v.w & head_mask);
  }
  lds_ready();                                       // the stage's memory is free for its loads
  static_assert(4 * D + 2 * 8 * D * 2 <= kStageBytes, "table and queries fit a stage");
  issue(std::integral_constant<int, kStages - 1>{}, kStages - 1, std::false_type{});

  // ---- state of the unit and of the split's units so far (lane: head `col` % 8, dims 16 d + 4 grp
  // + 0..3 of O, its own keys' part of the sum)
  f32x4 o[ND], o_run[kSolo ? 1 : ND];
  float m = -INFINITY, lsum = 0.0f, m_run = -INFINITY, l_run = 0.0f;
#pragma unroll
  for (int d = 0; d < ND; ++d) o[d] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};

  // LDS addresses: K fragment ss of tile t: row 16 t + col, chunk 4 ss + grp (fp8: 8 bytes at
  // 32 ss + 8 grp); V^T fragment d: bf16 rows 4 grp + (col / 4) of each tile, 8 bytes at dim 16 d +
  // 4 (col % 4); fp8 rows 4 grp + {0..3, 16..19}[col / 2], 8 bytes at dim 16 d + 8 (col % 2).
  const int kk = kFp8 ? 4 * grp + ((col >> 1) & 3) + 16 * (col >> 3) : 4 * grp + (col >> 2);
  const uint32_t k_lane = kFp8 ? col * RB + 16 * ((grp >> 1) ^ SW::k(col)) + 8 * (grp & 1) : col * RB + 16 * (grp ^ SW::k(col));
  const uint32_t v_lane = kFp8 ? SK * RB + kk * RB + 16 * SW::v(kk) + 8 * (col & 1)
                               : SK * RB + kk * RB + 16 * (((col & 3) >> 1) ^ SW::v(kk)) + 8 * (col & 1);

  const bool is_lo = col >= 8;
  // O of the unit: the sums over the weights' high parts and over their remainders
  auto unit_o = [&](int d) -> f32x4 {
    return (f32x4){add_ror8(o[d][0]), add_ror8(o[d][1]), add_ror8(o[d][2]), add_ror8(o[d][3])};
  };
  // O^T += V^T P^T over the keys of a stage's block
  auto add_values = [&](const lds_char* lds, int blk, const uint32_t (&pw)[2 * NTL]) {
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      const uint32_t row = blk * BK * RB;
      if constexpr (kFp8) {
        const i32x2 x = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2*)(lds + row + (v_lane ^ (uint32_t)(16 * d))));
        o[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(widen_fp8x8((uint32_t)x.x, (uint32_t)x.y)),
                                                       as_bf16x8(make_uint4(pw[0], pw[1], pw[2], pw[3])), o[d], 0, 0, 0);
      } else {
        const uint32_t at = row + (v_lane ^ (uint32_t)(32 * d));
        const i16x4 x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(lds + at));
        if constexpr (NTL == 2) {
          const i16x4 x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(lds + at + 16 * RB));
          const uint2 u0 = __builtin_bit_cast(uint2, x0), u1 = __builtin_bit_cast(uint2, x1);
          o[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(make_uint4(u0.x, u0.y, u1.x, u1.y)),
                                                         as_bf16x8(make_uint4(pw[0], pw[1], pw[2], pw[3])), o[d], 0, 0, 0);
        } else {
          const i16x4 p = __builtin_bit_cast(i16x4, make_uint2(pw[0], pw[1]));
          o[d] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x0, p, o[d], 0, 0, 0);
        }
      }
    }
  };
  // kFew, a row of a few keys: no rounding but the queries' is left in its result.  Scores are scaled before the
  // reference is taken from them (the largest weight is exactly 1) and the weights keep a third part,
  // which makes them exact: 16 keys 3.1e-6 -> 2.9e-6 off the 64-bit result, a single key's value as it is.
  // A copy of the loop, because the tests in it cost the others 6% (fp8 at head_dim 256).
  auto stage = [&](auto st, int i, auto few) {
    constexpr bool kFew = decltype(few)::value;
    // stage i has landed: the loads of the kStages - 1 later ones may be in flight
    __builtin_amdgcn_s_waitcnt(vm_wait((kStages - 1) * kLoads));
    asm volatile("" ::: "memory");
    uint4* mem = stage_mem(st);
    const lds_char* lds = (const lds_char*)(lds_void*)mem;
    const int key0 = k0 + i * SK;
    if (has_new && ctx >= key0 && ctx < key0 + SK) {          // the new token's rows (uniform)
      const int r = ctx - key0;
      if (lane < NCH) {
        mem[r * NCH + (lane ^ SW::k(r))] = new_k;
        mem[SK * NCH + r * NCH + (lane ^ SW::v(r))] = new_v;
      }
      __builtin_amdgcn_s_waitcnt(kLgkmWait);
      asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int blk = 0; blk < SK / BK; ++blk) {
      const int kb = key0 + blk * BK;
      f32x4 sc[NTL];
#pragma unroll
      for (int t = 0; t < NTL; ++t) {
        sc[t] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ss = 0; ss < NS; ++ss) {
          const uint32_t row = (blk * BK + 16 * t) * RB;
          uint4 kf;
          if constexpr (kFp8) {
            const u32x2 x = *reinterpret_cast<const lds_u32x2*>(lds + row + (k_lane ^ (uint32_t)(32 * ss)));
            kf = widen_fp8x8(x.x, x.y);
          } else {
            kf = __builtin_bit_cast(uint4, *reinterpret_cast<const lds_u32x4*>(lds + row + (k_lane ^ (uint32_t)(64 * ss))));
          }
          sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(kf), as_bf16x8(q[ss]), sc[t], 0, 0, 0);
        }
      }
      // lane: head col % 8 (columns 8-15 repeat 0-7 once hi and lo are added), keys kb + 16 t +
      // 4 grp + e
#pragma unroll
      for (int t = 0; t < NTL; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[t][e] = add_ror8(sc[t][e]);
      if (kb < lo || kb + BK > k1) {
#pragma unroll
        for (int t = 0; t < NTL; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int key = kb + 16 * t + 4 * grp + e;
            sc[t][e] = (key >= lo && key < k1) ? sc[t][e] : -INFINITY;
          }
      }
      if constexpr (kFew) {
#pragma unroll
        for (int t = 0; t < NTL; ++t) sc[t] *= a.scale_log2;
      }
      const float scale = kFew ? 1.0f : a.scale_log2;
      float mx = -INFINITY;
#pragma unroll
      for (int t = 0; t < NTL; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) mx = fmaxf(mx, sc[t][e]);
      const float mx2 = max_over_groups(mx) * scale;
      const bool raised = mx2 > m;
      if (__builtin_amdgcn_ballot_w64(raised) != 0) {
        const float alpha = raised ? __builtin_amdgcn_exp2f(m - mx2) : 1.0f;
        m = raised ? mx2 : m;
        lsum *= alpha;
#pragma unroll
        for (int d = 0; d < ND; ++d) o[d] *= alpha;
      }
      const float m_ref = m == -INFINITY ? 0.0f : m;          // no key seen yet: every p is 0
      // weights as bf16 pairs: their high parts in columns 0-7, the remainders in columns 8-15
      uint32_t pw[2 * NTL];
#pragma unroll
      for (int t = 0; t < NTL; ++t)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[t][e], scale, -m_ref));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[t][e + 1], scale, -m_ref));
          lsum += p0;
          lsum += p1;
          if constexpr (kFew) {
            sc[t][e] = p0;
            sc[t][e + 1] = p1;
          }
          const bf16x2 h = __builtin_convertvector((f32x2){p0, p1}, bf16x2);
          const uint32_t lw = pack_bf16_rne(p0 - (float)h.x, p1 - (float)h.y);
          pw[2 * t + e / 2] = is_lo ? lw : __builtin_bit_cast(uint32_t, h);
        }
      add_values(lds, blk, pw);
      if constexpr (kFew) {
        // what hi and lo leave of a weight, exactly (columns 0-7)
#pragma unroll
        for (int t = 0; t < NTL; ++t)
#pragma unroll
          for (int e = 0; e < 4; e += 2) {
            const float p0 = sc[t][e], p1 = sc[t][e + 1];
            const bf16x2 h = __builtin_convertvector((f32x2){p0, p1}, bf16x2);
            const float r0 = p0 - (float)h.x, r1 = p1 - (float)h.y;
            const bf16x2 lw = __builtin_convertvector((f32x2){r0, r1}, bf16x2);
            pw[2 * t + e / 2] = is_lo ? 0u : pack_bf16_rne(r0 - (float)lw.x, r1 - (float)lw.y);
          }
        add_values(lds, blk, pw);
      }
    }
    // the stage's reads have returned: its memory takes stage i + kStages
    __builtin_amdgcn_s_waitcnt(kLgkmWait);
    asm volatile("" ::: "memory");
    issue(st, i + kStages, std::false_type{});
    if constexpr (!kSolo) {
      if (((i + 1) % kUnitStages == 0 && i + 1 < 4 * kUnitStages) || i + 1 == n_stages) {   // end of a unit
        const float lu = sum_over_groups(lsum);
        if (i < kUnitStages) {
          m_run = m;
          l_run = lu;
#pragma unroll
          for (int d = 0; d < ND; ++d) o_run[d] = unit_o(d);
        } else {
          const float m_new = fmaxf(m_run, m);
          const float f_me = merge_factor(m_run, m_new);
          const float f_o = merge_factor(m, m_new);
          l_run = fmaf(l_run, f_me, lu * f_o);
          m_run = m_new;
#pragma unroll
          for (int d = 0; d < ND; ++d) {
            const f32x4 ou = unit_o(d);
#pragma unroll
            for (int e = 0; e < 4; ++e) o_run[d][e] = fmaf(o_run[d][e], f_me, ou[e] * f_o);
          }
        }
        m = -INFINITY;
        lsum = 0.0f;
#pragma unroll
        for (int d = 0; d < ND; ++d) o[d] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
      }
    }
  };
  auto walk = [&](auto few) {
    for (int i = 0; i < n_stages; i += kStages) {
      stage(S0{}, i, few);
      if (i + 1 < n_stages) stage(S1{}, i + 1, few);
      if constexpr (kStages > 2) {
        if (i + 2 < n_stages) stage(S2{}, i + 2, few);
      }
    }
  };
  if (n_keys - lo <= kFewKeys)
    walk(std::true_type{});
  else
    walk(std::false_type{});

  // the empty loads past the last stage write LDS too: none may outlive the wave
  __builtin_amdgcn_s_waitcnt(vm_wait(0));
  // ---- the wave's partial, or the output itself when the row has one split
  if constexpr (kSolo) {
    const float lu = sum_over_groups(lsum);
#pragma unroll
    for (int d = 0; d < ND; ++d) o[d] = unit_o(d);
    if (col < G && n_keys - base <= kUnit) {         // the row's only unit
      float* op = a.out + (head0 + col) * D + 4 * grp;
#pragma unroll
      for (int d = 0; d < ND; ++d)
        *reinterpret_cast<f32x4*>(op + 16 * d) = (f32x4){o[d][0] / lu, o[d][1] / lu, o[d][2] / lu, o[d][3] / lu};
    } else if (col < G) {
      const int64_t pidx = (head0 + col) * unit_slots(a.n_split_max, a.n_shared_split) + unit_slot(s, a.n_shared_split) + unit0;
#pragma unroll
      for (int d = 0; d < ND; ++d) *reinterpret_cast<f32x4*>(a.part_acc + pidx * D + 16 * d + 4 * grp) = o[d];
      if (grp == 0) *reinterpret_cast<float2*>(a.part_ml + pidx * 2) = make_float2(m, lu);
    }
  } else if (col < G) {
    if (n_split == 1) {
      float* op = a.out + (head0 + col) * D + 4 * grp;
#pragma unroll
      for (int d = 0; d < ND; ++d)
        *reinterpret_cast<f32x4*>(op + 16 * d) = (f32x4){o_run[d][0] / l_run, o_run[d][1] / l_run, o_run[d][2] / l_run, o_run[d][3] / l_run};
      return;
    }
    const int64_t pidx = (head0 + col) * a.n_split_max + s;
#pragma unroll
    for (int d = 0; d < ND; ++d) *reinterpret_cast<f32x4*>(a.part_acc + pidx * D + 16 * d + 4 * grp) = o_run[d];
    if (grp == 0) *reinterpret_cast<float2*>(a.part_ml + pidx * 2) = make_float2(m_run, l_run);
  }
}

}  // namespace

template <typename T, bool kSolo, int kStages>
hipError_t launch_decode_mfma_t(const DecodeArgs& a, hipStream_t stream) {
  const int64_t n_wg = decode_items(a) * (kSolo ? 4 : 1);
  const dim3 grid((unsigned)n_wg);
  switch (a.D) {
    case 64: decode_mfma_kernel<T, 64, kSolo, 2><<<grid, 64, 0, stream>>>(a); break;
    case 128: decode_mfma_kernel<T, 128, kSolo, sizeof(T) == 2 ? kStages : 2><<<grid, 64, 0, stream>>>(a); break;
    case 256: decode_mfma_kernel<T, 256, kSolo, kStages><<<grid, 64, 0, stream>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Stages in flight of a wave per split.  Rows of at least 256 bytes (16 KiB stages): three, which leave room for
// three waves on a CU, 768 in all, and run faster than two with five (16 sequences x 4.6k keys at head_dim 256:
// bf16 117 -> 105 us, fp8 72 -> 66).  A launch of a little more than one or two rounds of those pays for a whole
// round more, and takes two: us at head_dim 256 with three / two stages, bf16 and fp8,
//   792 splits   95 / 78,  62 / 46      1,224   108 / 127,  66 / 83
//   1,008       102 / 88,  64 / 55      1,440   124 / 138,  72 / 90
//   1,728       162 / 157, 97 / 94      2,016   173 / 178, 101 / 107
//   2,592       232 / 230, 134 / 138    3,168   289 / 291, 165 / 170
// Four stages leave two waves a CU: 168 and 125 at 1,728.  Two waves that share a split, half each, were no
// faster either (158, 100).  Shorter rows have 8 KiB stages, two of them: ten waves a CU, whose 32-key blocks, one
// after the other, are what bounds them (64-byte rows, 8 heads x 64 sequences over 30k keys: 487 us with
// 16 KiB stages, 328).
template <typename T>
hipError_t launch_decode_type(const DecodeArgs& a, hipStream_t stream) {
  if (a.solo) return launch_decode_mfma_t<T, true, 2>(a, stream);
  constexpr int64_t kRound = 3 * 256;
  const int64_t n = decode_items(a), over = n % kRound;
  const bool two = n > kRound && n < 3 * kRound && over > 0 && over <= kRound / 3;
  return two ? launch_decode_mfma_t<T, false, 2>(a, stream) : launch_decode_mfma_t<T, false, 3>(a, stream);
}

hipError_t launch_decode_mfma(const DecodeArgs& a, int dtype, hipStream_t stream) {
  if (dtype == kDtypeBf16) return launch_decode_type<uint16_t>(a, stream);
  if (dtype == kDtypeFp8) return launch_decode_type<uint8_t>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace kvg
