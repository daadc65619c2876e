// Grouped-query decode attention of fp32 caches on the vector ALUs (one new token per sequence), split
// over keys ("split-K"); and the kernels that combine the split partials of every cache type.
//
// Work item = (layer, sequence, row, KV head g, split s).  A split is a fixed logical key range of
// the row's visible keys; the split plan is a function of the row's own length and window only.
// One 256-thread workgroup per work item:
//   - teams of TL lanes (16) each own every NT-th key of the split (key k0 + team + NT i); lane
//     tl of a team holds 16-byte chunks tl, tl + TL, ... of the D-wide K and V rows, so a team
//     reads whole rows with 16-byte loads, and each team keeps up to four keys' rows in flight
//     while it computes.
//   - q for the `group` query heads that share KV head g sits in registers.
//   - per key: partial dot products, an xor butterfly inside the team (every lane ends
//     with identical bits because each step adds the same two values), then an online
//     softmax update of the team's running (reference m, sum l, weighted V acc)
//     with exp2 of pre-scaled scores; the reference m is raised only when a score exceeds
//     it by more than 2^8, so most keys cost one exp2 and one FMA per element.
//   - the team states are merged with a fixed xor tree inside each wavefront, then waves
//     0..3 in order through LDS.
// Splits are combined in ascending split order.  Nothing depends on physical page ids or
// on how many rows/sequences share the launch, which is what makes the graft path and the
// fresh path produce the same bytes.
#include "kvg_device.h"
#include "kvg_launch.h"
#include "kvg_rows.h"

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace kvg {

namespace {

constexpr int kThreads = 256;
constexpr float kRescale = 8.0f;     // lazy-rescale threshold of the running reference (log2 units)

// Cached K/V rows are read once per call: streaming (nontemporal) loads.  Measured on the
// 12B-class decode (1.83 GB per call over random pages): 326 -> 300 us per call.
typedef unsigned int u32x4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld16_stream(const void* p) {
  const u32x4v v = __builtin_nontemporal_load(reinterpret_cast<const u32x4v*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
// c ? a : b per 32-bit component (a select of uint4 lvalues would select addresses and
// keep the operands in memory)
__device__ __forceinline__ uint4 sel4(bool c, const uint4& a, const uint4& b) {
  return make_uint4(c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z, c ? a.w : b.w);
}
struct Soft {
  float m, l;
};

// Sum over the TL lanes of a team (TL = 4, 8 or 16 consecutive lanes) with DPP moves:
// partners lane ^ 1 and lane ^ 2 inside each quad, then the mirrored lane inside each half
// row and row.  After the quad steps all lanes of a quad hold the same bits, so the mirror
// steps pair the same two values an xor-4 / xor-8 butterfly would; every step adds the same
// two values in both partner lanes, so the whole team ends with identical bits.
template <int TL>
__device__ __forceinline__ float team_sum(float x) {
  static_assert(TL == 4 || TL == 8 || TL == 16, "team width");
  x += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, true));
  x += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, true));
  if constexpr (TL >= 8)
    x += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x141, 0xF, 0xF, true));
  if constexpr (TL >= 16)
    x += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x140, 0xF, 0xF, true));
  return x;
}

// Page ids of a split's keys (at most kSplit / kPage + 1 pages, a window's split starting
// inside a page): lane i of every wave holds the page of logical page `first` + i, read
// once, so the key-row loads never wait on a block-table read.  The teams of one wave
// always read keys of the same logical page at a time, so the page of a key is taken with a
// lane read.
struct SplitPages {
  static_assert(kSplit / kPage + 1 <= 64, "a split's pages must fit a wave");
  int32_t pg;
  int base;
  // the block-table entries of the 64 pages from page `first` on, clamped to the table's
  // n_table entries (entries past the context are never used)
  __device__ __forceinline__ void init(const int32_t* bt, int first, int n_table, int lane) {
    base = first;
    pg = bt[min(base + lane, n_table - 1)];
  }
  __device__ __forceinline__ int32_t page_of(int j) const {
    const int i = __builtin_amdgcn_readfirstlane(j / kPage - base);
    return __builtin_amdgcn_readlane(pg, i);
  }
};

template <int D, int G>
struct SplitWorker {
  static constexpr int CH = Elem<float>::kPerVec; // elements per 16-byte chunk
  static constexpr int NCH = D / CH;              // chunks per row
  static constexpr int TL = NCH < 16 ? NCH : 16;  // lanes per key ("team")
  static constexpr int CPL = NCH / TL;            // chunks per lane
  static constexpr int EPL = CPL * CH;            // elements per lane
  static constexpr int NT = kThreads / TL;        // teams per workgroup
  // key pairs in flight per team (the consumption order, and so the arithmetic, does not
  // depend on it)
  static constexpr int kPairs = 2;
  static_assert(CPL >= 1 && (64 % TL) == 0 && TL >= 4, "unsupported head_dim");
  // a wave's teams never straddle a logical page: (64 / TL) teams per wave divide 16
  static_assert(kThreads / TL >= kPage, "teams per workgroup");

  struct Row {
    uint4 k[CPL], v[CPL];
    bool ok;
    bool lds;          // the new decode token: rows come from LDS when consumed
  };

  float q[G][EPL];
  float acc[G][EPL];
  Soft st[G];
  int tl, team, lane, wave;
  const uint4* lds_k = nullptr;   // the new token's K/V rows (16-byte chunks) in LDS
  const uint4* lds_v = nullptr;

  __device__ __forceinline__ void init() {
    lane = threadIdx.x & 63;
    wave = threadIdx.x >> 6;
    tl = lane % TL;
    team = threadIdx.x / TL;
#pragma unroll
    for (int h = 0; h < G; ++h) {
      st[h].m = -INFINITY;
      st[h].l = 0.0f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[h][e] = 0.0f;
    }
  }

  // Query chunk j of this lane is chunk q_chunk(j) of the row's.
  __device__ __forceinline__ int q_chunk(int j) const { return tl + TL * j; }
  __device__ __forceinline__ void set_q(int h, int j, const uint4& v) {
    q[h][j * 4 + 0] = __uint_as_float(v.x);
    q[h][j * 4 + 1] = __uint_as_float(v.y);
    q[h][j * 4 + 2] = __uint_as_float(v.z);
    q[h][j * 4 + 3] = __uint_as_float(v.w);
  }

  // Branches in the consume functions are uniform over the wavefront (ballots), so the
  // loads of later rows stay in flight across them.  A key that is not ok contributes
  // p = 0: its row is a visible key's row (a key past the split loads key k1 - 1, one
  // below the window its first; the decode's new token is taken from LDS), so 0 * V adds nothing.  Only a block-table
  // entry outside the pool (whose outputs are unspecified) can bring other bytes.
  __device__ __forceinline__ void fix_row(Row& rw) {
    if (__builtin_amdgcn_ballot_w64(rw.lds) != 0) {
#pragma unroll
      for (int i = 0; i < CPL; ++i) {
        const uint4 lk = lds_k[tl + TL * i], lv = lds_v[tl + TL * i];
        rw.k[i] = sel4(rw.lds, lk, rw.k[i]);
        rw.v[i] = sel4(rw.lds, lv, rw.v[i]);
      }
    }
  }

  // the key's scores for the G heads (log2 units), -inf for a key that is not ok
  __device__ __forceinline__ void scores(const Row& rw, float scale_log2, float (&s2)[G]) {
    float sc[G];
#pragma unroll
    for (int h = 0; h < G; ++h) sc[h] = 0.0f;
#pragma unroll
    for (int i = 0; i < CPL; ++i)
#pragma unroll
      for (int e = 0; e < CH; ++e) {
        const float kf = Elem<float>::get(rw.k[i], e);
#pragma unroll
        for (int h = 0; h < G; ++h) sc[h] = fmaf(q[h][i * CH + e], kf, sc[h]);
      }
#pragma unroll
    for (int h = 0; h < G; ++h) s2[h] = rw.ok ? team_sum<TL>(sc[h]) * scale_log2 : -INFINITY;
  }

  // lazy rescale: the running reference only moves when a score exceeds it by more than
  // kRescale, so p = exp2(s2 - m) stays <= 2^kRescale; lanes that keep their reference
  // multiply by exactly 1
  __device__ __forceinline__ void raise_to(int h, float mx) {
    const bool raise = mx > st[h].m + kRescale;
    if (__builtin_amdgcn_ballot_w64(raise) != 0) {
      const float alpha = raise ? ((st[h].m == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(st[h].m - mx)) : 1.0f;
      st[h].m = raise ? mx : st[h].m;
      st[h].l *= alpha;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[h][e] *= alpha;
    }
  }

  // one key, p and the weighted V in fp32
  __device__ __forceinline__ void consume(Row& rw, float scale_log2) {
    fix_row(rw);
    float s2[G];
    scores(rw, scale_log2, s2);
#pragma unroll
    for (int h = 0; h < G; ++h) {
      raise_to(h, s2[h]);
      const float p = rw.ok ? __builtin_amdgcn_exp2f(s2[h] - st[h].m) : 0.0f;
      st[h].l += p;
#pragma unroll
      for (int i = 0; i < CPL; ++i) {
#pragma unroll
        for (int e = 0; e < CH; ++e) acc[h][i * CH + e] = fmaf(p, Elem<float>::get(rw.v[i], e), acc[h][i * CH + e]);
      }
    }
  }

  // Keys k0 + team, k0 + team + NT, ... below k1, in stages of two keys with kPairs stages
  // (2 kPairs rows) in flight per team.  load(j, row) fills a row for a key j < k1.  Every
  // fetch is unconditional, so the loads stay in flight across the loop's back edge: a key
  // past k1 loads the row of key k1 - 1 (the same L2-resident row for every team) and is
  // marked not ok, which consume() turns into an exact no-op.  prologue() runs after the
  // first stages are in flight, so per-workgroup setup overlaps their latency; the queries
  // must be set by the time it returns.
  template <class Load, class Prologue>
  __device__ __forceinline__ void run(int k0, int k1, float scale_log2, Load load, Prologue prologue) {
    auto fetch = [&](int j, Row& rw) {
      const bool in = j < k1;
      load(in ? j : k1 - 1, rw);
      rw.ok = rw.ok && in;
    };
    const int n_it = (k1 - k0 + NT - 1) / NT;     // keys per team, rounded up
    constexpr int R = 2 * kPairs;                 // rows in flight per team
    Row rows[R];
    int j = k0 + team;
#pragma unroll
    for (int r = 0; r < R; ++r) fetch(j + r * NT, rows[r]);
    __builtin_amdgcn_sched_barrier(0);
    prologue();
    // Keys are consumed in order, a pair at a time; each pair's rows are refetched R keys
    // ahead as soon as they are consumed.  The scheduling barriers keep each stage's loads
    // where they are issued here (the scheduler would otherwise sink them to the end of the
    // body to shorten live ranges).
    for (int it = 0; it < n_it; it += R) {
#pragma unroll
      for (int p = 0; p < kPairs; ++p) {
        consume(rows[2 * p], scale_log2);
        consume(rows[2 * p + 1], scale_log2);
        __builtin_amdgcn_sched_barrier(0);
        fetch(j + (R + 2 * p) * NT, rows[2 * p]);
        fetch(j + (R + 2 * p + 1) * NT, rows[2 * p + 1]);
        __builtin_amdgcn_sched_barrier(0);
      }
      j += R * NT;
    }
  }

  // Merge the teams of each wavefront (xor tree over lanes with equal tl) and leave each
  // wave's state in LDS: s_acc[wave][h][d], s_ml[wave][h] = (m, l).
  __device__ __forceinline__ void to_lds(float (*s_acc)[G][D], float (*s_ml)[G][2]) {
#pragma unroll
    for (int mask = TL; mask < 64; mask <<= 1) {
#pragma unroll
      for (int h = 0; h < G; ++h) {
        const float m_o = __shfl_xor(st[h].m, mask);
        const float l_o = __shfl_xor(st[h].l, mask);
        const float m_new = fmaxf(st[h].m, m_o);
        const float f_me = merge_factor(st[h].m, m_new);
        const float f_o = merge_factor(m_o, m_new);
        st[h].l = st[h].l * f_me + l_o * f_o;
        st[h].m = m_new;
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
          const float a_o = __shfl_xor(acc[h][e], mask);
          acc[h][e] = acc[h][e] * f_me + a_o * f_o;
        }
      }
    }
    if (lane < TL) {
#pragma unroll
      for (int h = 0; h < G; ++h) {
#pragma unroll
        for (int i = 0; i < CPL; ++i) {
#pragma unroll
          for (int e = 0; e < CH; ++e) s_acc[wave][h][(tl + TL * i) * CH + e] = acc[h][i * CH + e];
        }
        if (lane == 0) {
          s_ml[wave][h][0] = st[h].m;
          s_ml[wave][h][1] = st[h].l;
        }
      }
    }
  }
};

// The split's state for (head h, element d): waves 0..3 merged in order.
template <int G, int D>
__device__ __forceinline__ void wave_merge(const float (*s_acc)[G][D], const float (*s_ml)[G][2], int h, int d,
                                           float& m, float& lsum, float& o) {
  m = s_ml[0][h][0];
  lsum = s_ml[0][h][1];
  o = s_acc[0][h][d];
#pragma unroll
  for (int wv = 1; wv < 4; ++wv) {
    const float m_o = s_ml[wv][h][0];
    const float m_new = fmaxf(m, m_o);
    const float f_me = merge_factor(m, m_new);
    const float f_o = merge_factor(m_o, m_new);
    lsum = lsum * f_me + s_ml[wv][h][1] * f_o;
    o = o * f_me + s_acc[wv][h][d] * f_o;
    m = m_new;
  }
}

// Final value of one output element from the splits' (m, l) pairs and weighted-V values
// (acc[s * acc_stride]), combined in ascending split order.
// Splits are taken U (eight unless the caller knows fewer) at a time with every load issued
// before its use: indices past the last split re-read the last one (a repeat changes no
// maximum) and are not added.  The sums run over the splits in ascending order whatever
// the unrolling, so every path that combines the same partials gives the same bytes.
template <int U = 8>
__device__ __forceinline__ float combine_splits(const float* ml, const float* acc, int64_t acc_stride, int n_split) {
  float m = -INFINITY;
  for (int s0 = 0; s0 < n_split; s0 += U) {
    float mv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) mv[u] = ml[2 * min(s0 + u, n_split - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) m = fmaxf(m, mv[u]);
  }
  float lsum = 0.0f, o = 0.0f;
  for (int s0 = 0; s0 < n_split; s0 += U) {
    float2 pv[U];
    float av[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = min(s0 + u, n_split - 1);
      pv[u] = *reinterpret_cast<const float2*>(ml + 2 * s);
      av[u] = acc[s * acc_stride];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float f = merge_factor(pv[u].x, m);
      const bool in = s0 + u < n_split;
      lsum = in ? fmaf(pv[u].y, f, lsum) : lsum;
      o = in ? fmaf(av[u], f, o) : o;
    }
  }
  return o / lsum;
}

// ------------------------------------------------------------------------------------
// Decode: the split kernel rotates its queries from the raw input (angles in fp64 once per
// workgroup) and the last split's workgroup appends the new token's K/V for its KV head
// (written to the cache and kept in LDS for its own use).  A context that fits one split
// is finished in place; longer ones are combined by decode_merge_kernel in ascending split
// order.  (Combining in the last-arriving workgroup would need a device-scope release per
// workgroup, an L2 write-back on this chip that cost more than the second launch.)
template <int D, int G>
__global__ __launch_bounds__(kThreads) void decode_kernel(const DecodeArgs a) {
  using W = SplitWorker<D, G>;
  using R = float;                                  // raw rows and cache rows
  using T = float;
  constexpr int NCH = W::NCH;                       // 16-byte chunks of a row
  constexpr int ER = Elem<R>::kPerVec;
  constexpr int NCHR = NCH;
  // Sequence index fastest.  When the sequences share leading pages (a shared window,
  // shared_order), runs of 64 consecutive work items go to one XCD (workgroups are dealt
  // to the 8 XCDs in turn), so the sequences reading the same keys do so at about the same
  // time through one L2: 32 sequences over a shared 32k-token window decode 8 steps in
  // 212 instead of 367 ms.  Private pages keep the plain order, which measured 5% faster
  // there.  The arithmetic of a work item does not depend on the order.
  int64_t w = blockIdx.x;
  if (a.shared_order) {
    constexpr int64_t CH = 64;
    const int64_t full = (int64_t)gridDim.x / (8 * CH) * (8 * CH);
    if (w < full) {
      const int64_t g8 = w / 8;
      w = ((g8 / CH) * 8 + w % 8) * CH + g8 % CH;
    }
  }
  const DecodeItem item = decode_item(a, w);
  const int b = item.b, si = item.si, g = item.g, l = item.l;

  const int tid = threadIdx.x;
  constexpr int QCH = G * NCHR;                     // 16-byte chunks of the group's raw q
  constexpr int QPT = (QCH + kThreads - 1) / kThreads;
  const int64_t tok = (int64_t)l * a.batch + b;   // the step's raw row index

  // Requested before the context length is known, which they do not depend on: the
  // split's block-table entries, then the step's raw rows (the prologue waits for these
  // alone, the memory counter being in order; every thread loads one 16-byte chunk, indices
  // clamped; the new token's k and v are read by every split, used by the last).
  const int32_t* bt = a.block_tables + (int64_t)b * a.max_pages;
  const int win = layer_window(a, l);
  // the grid holds no shared split (the shared-split kernel's): a full-attention layer's
  // items start after them
  const int s = (win == 0 ? a.n_shared_split : 0) + si;
  SplitPages sp;
  if (win == 0) sp.init(bt, s * (kSplit / kPage), a.max_pages, tid & 63);   // split s = keys [512 s, ...)
  uint4 rq[QPT];
  const R* qraw = reinterpret_cast<const R*>(a.q_raw) + (tok * a.Hq + (int64_t)g * G) * D;
#pragma unroll
  for (int r = 0; r < QPT; ++r) rq[r] = ld16(qraw + min(tid + r * kThreads, QCH - 1) * ER);
  const R* kraw = reinterpret_cast<const R*>(a.k_raw) + (tok * a.Hkv + g) * D;
  const R* vraw = reinterpret_cast<const R*>(a.v_raw) + (tok * a.Hkv + g) * D;
  const uint4 rk = ld16(kraw + min(tid, NCHR - 1) * ER);
  const uint4 rv = ld16(vraw + min(tid, NCHR - 1) * ER);
  __builtin_amdgcn_sched_barrier(0);              // keep these loads ahead of the key rows

  const int ctx = a.ctx_lens[b];
  if (ctx < 0 || ctx > a.max_ctx_len) return;
  const int n_keys = ctx + 1;                     // the new token is key ctx
  const int lo = window_start(win, n_keys);
  const int n_split = split_count(n_keys, lo);
  if (s >= n_split) return;
  const int k0 = lo + s * kSplit;                 // the split's keys [k0, k1)
  const int k1 = min(k0 + kSplit, n_keys);
  const int kb = k0 & ~(kPage - 1);               // teams start at the page holding k0
  const bool last_split = s == n_split - 1;
  if (win != 0) sp.init(bt, kb / kPage, a.max_pages, tid & 63);

  __shared__ float cs[2 * kMaxHalfDim];
  __shared__ uint4 new_k[NCH], new_v[NCH];
  __shared__ uint4 raw_q[QCH], raw_k[NCHR], raw_v[NCHR];
  __shared__ float s_acc[4][G][D];
  __shared__ float s_ml[4][G][2];

  const int64_t lbase = (int64_t)(a.layer0 + l) * a.layer_elems;
  T* kpool = reinterpret_cast<T*>(a.k_pool) + lbase;
  T* vpool = reinterpret_cast<T*>(a.v_pool) + lbase;
  const int64_t pos = a.start_pos[b] + ctx;       // absolute position of the new token

  W wk;
  wk.init();
  wk.lds_k = new_k;
  wk.lds_v = new_v;

  // The new token (key ctx) is not in the cache yet when its row is requested: its slot's
  // old bytes are loaded like any row (in bounds, discarded) and the key is consumed from
  // LDS, so no branch depends on the key.
  auto load = [&](int j, typename W::Row& rw) {
    const int32_t page = sp.page_of(j);
    const bool valid = page >= 0 && page < a.n_pages;
    rw.lds = j == ctx;
    rw.ok = rw.lds || (valid && j >= k0);
    const int64_t roff = (((int64_t)(valid ? page : 0) * a.Hkv + g) * kPage + (max(j, k0) % kPage)) * D;
#pragma unroll
    for (int i = 0; i < W::CPL; ++i) rw.k[i] = ld16_stream(kpool + roff + (wk.tl + W::TL * i) * W::CH);
#pragma unroll
    for (int i = 0; i < W::CPL; ++i) rw.v[i] = ld16_stream(vpool + roff + (wk.tl + W::TL * i) * W::CH);
  };
  // runs while the first key rows are in flight: rotation table, the new token's K/V
  // (last split: rotated K, written to the cache and kept in LDS), the rotated queries
  auto prologue = [&] {
    for (int p = tid; p < D / 2; p += kThreads) {
      double sn, cn;
      sincos((double)pos * a.theta[p], &sn, &cn);
      cs[2 * p] = (float)cn;
      cs[2 * p + 1] = (float)sn;
    }
#pragma unroll
    for (int r = 0; r < QPT; ++r)
      if (tid + r * kThreads < QCH) raw_q[tid + r * kThreads] = rq[r];
    if (tid < NCHR) {
      raw_k[tid] = rk;
      raw_v[tid] = rv;
    }
    __syncthreads();
    // the new token's V in the cache dtype (every split: a row equal to key ctx is taken
    // from LDS when it is consumed, which only the last split does)
    for (int c = tid; c < NCH; c += kThreads)
      new_v[c] = storage_chunk<D>(reinterpret_cast<const float*>(raw_v), c, false, a.pairing, cs);
    if (last_split) {
      const int32_t page = sp.page_of(ctx);
      const bool ok = page >= 0 && page < a.n_pages;
      const int64_t roff = (((int64_t)(ok ? page : 0) * a.Hkv + g) * kPage + (ctx % kPage)) * D;
      for (int c = tid; c < NCH; c += kThreads) {
        const uint4 kc = storage_chunk<D>(reinterpret_cast<const float*>(raw_k), c, true, a.pairing, cs);
        new_k[c] = kc;
        if (ok) {
          st16(kpool + roff + c * W::CH, kc);
          st16(vpool + roff + c * W::CH, new_v[c]);       // written by this thread above
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int j = 0; j < W::CPL; ++j)
        wk.set_q(h, j, storage_chunk<D>(reinterpret_cast<const float*>(raw_q) + h * D, wk.q_chunk(j), true, a.pairing, cs));
  };
  wk.run(kb, k1, a.scale_log2, load, prologue);

  wk.to_lds(s_acc, s_ml);
  __syncthreads();

  const int64_t head0 = tok * a.Hq + (int64_t)g * G;     // output row of head 0 of the group
  if (n_split == 1) {
    for (int t = tid; t < G * D; t += kThreads) {
      const int h = t / D, d = t - (t / D) * D;
      alignas(8) float ml[2];
      float o;
      wave_merge<G, D>(s_acc, s_ml, h, d, ml[0], ml[1], o);
      a.out[(head0 + h) * D + d] = combine_splits(ml, &o, 0, 1);
    }
    return;
  }

  // publish this split's partial; decode_merge_kernel combines the splits
  for (int t = tid; t < G * D; t += kThreads) {
    const int h = t / D, d = t - (t / D) * D;
    float m, lsum, o;
    wave_merge<G, D>(s_acc, s_ml, h, d, m, lsum, o);
    const int64_t pidx = (head0 + h) * a.n_split_max + s;
    a.part_acc[pidx * D + d] = o;
    if (d == 0) {
      a.part_ml[pidx * 2] = m;
      a.part_ml[pidx * 2 + 1] = lsum;
    }
  }
}

// Combine the split partials of every (layer, sequence, query head) row whose context
// needed more than one split, in ascending split order.
__global__ __launch_bounds__(kThreads) void decode_merge_kernel(const DecodeArgs a) {
  const int64_t row_head = blockIdx.x;            // (layer, batch, q head)
  const int b = (int)((row_head / a.Hq) % a.batch);
  const int l = (int)(row_head / ((int64_t)a.Hq * a.batch));
  constexpr int U = 16;
  if (a.n_split_max <= U && a.D <= kThreads) {
    // One memory round trip: the partials of every split the workspace holds are requested
    // together with the context length (in bounds; those of splits the row does not use
    // are not added), then combined exactly as combine_splits does.
    const float* ml = a.part_ml + row_head * a.n_split_max * 2;
    const float* acc = a.part_acc + row_head * a.n_split_max * a.D;
    const int d = min((int)threadIdx.x, a.D - 1);
    float2 pv[U];
    float av[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = min(u, a.n_split_max - 1);
      pv[u] = *reinterpret_cast<const float2*>(ml + 2 * s);
      av[u] = acc[s * a.D + d];
    }
    const int ctx = a.ctx_lens[b];
    if (ctx < 0 || ctx > a.max_ctx_len) return;
    const int win = layer_window(a, l);
    const int n_split = split_count(ctx + 1, window_start(win, ctx + 1));
    if (n_split == 1 && !(win == 0 && a.n_shared_split > 0)) return;   // written by the split kernel
    float m = -INFINITY;
#pragma unroll
    for (int u = 0; u < U; ++u) m = (u < n_split) ? fmaxf(m, pv[u].x) : m;
    float lsum = 0.0f, o = 0.0f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float f = merge_factor(pv[u].x, m);
      const bool in = u < n_split;
      lsum = in ? fmaf(pv[u].y, f, lsum) : lsum;
      o = in ? fmaf(av[u], f, o) : o;
    }
    if ((int)threadIdx.x < a.D) a.out[row_head * a.D + threadIdx.x] = o / lsum;
    return;
  }
  const int ctx = a.ctx_lens[b];
  if (ctx < 0 || ctx > a.max_ctx_len) return;
  const int win = layer_window(a, l);
  const int n_split = split_count(ctx + 1, window_start(win, ctx + 1));
  if (n_split == 1 && !(win == 0 && a.n_shared_split > 0)) return;     // written by the split kernel
  const float* ml = a.part_ml + row_head * a.n_split_max * 2;
  const float* acc = a.part_acc + row_head * a.n_split_max * a.D;
  constexpr int kLdsSplits = 2048;
  if (n_split <= kLdsSplits) {
    // Many splits of many rows: the (reference, sum) pairs are staged in LDS by the whole workgroup in
    // one round trip, and each lane requests 16 splits' values at a time; the arithmetic and its
    // order are combine_splits' own.
    __shared__ float s_ml[2 * kLdsSplits];
    for (int t = threadIdx.x; t < 2 * n_split; t += kThreads) s_ml[t] = ml[t];
    __syncthreads();
    float m = -INFINITY;
    for (int s = 0; s < n_split; ++s) m = fmaxf(m, s_ml[2 * s]);
    for (int d = threadIdx.x; d < a.D; d += kThreads) {
      float lsum = 0.0f, o = 0.0f;
      for (int s0 = 0; s0 < n_split; s0 += U) {
        float av[U];
#pragma unroll
        for (int u = 0; u < U; ++u) av[u] = acc[min(s0 + u, n_split - 1) * a.D + d];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int s = min(s0 + u, n_split - 1);
          const float f = merge_factor(s_ml[2 * s], m);
          const bool in = s0 + u < n_split;
          lsum = in ? fmaf(s_ml[2 * s + 1], f, lsum) : lsum;
          o = in ? fmaf(av[u], f, o) : o;
        }
      }
      a.out[row_head * a.D + d] = o / lsum;
    }
    return;
  }
  for (int d = threadIdx.x; d < a.D; d += kThreads)
    a.out[row_head * a.D + d] = combine_splits(ml, acc + d, a.D, n_split);
}

// Combine of rows with many splits, or (kSolo, DecodeArgs.solo) with four partials per split: the
// units of a split merged in order, then the splits in ascending order, combine_splits' own
// arithmetic.  A workgroup per (layer, sequence, query head): the splits' (reference, sum) pairs
// and weights are worked out once, in LDS; the lane groups then bring kMergeChunk splits' values
// at a time (every partial requested at once), and one lane per element sums them in order.
constexpr int kMergeChunk = 32;
// kBeside: (kSolo) beside shared splits, which have one partial.
template <bool kSolo, int kMergeThreads, bool kBeside = false>
__global__ __launch_bounds__(kMergeThreads) void merge_splits_kernel(const DecodeArgs a) {
  constexpr int U = kSolo ? 4 : 1;                         // partials per split
  const int64_t row_head = blockIdx.x;
  const int b = (int)((row_head / a.Hq) % a.batch);
  const int l = (int)(row_head / ((int64_t)a.Hq * a.batch));
  const int D = a.D;
  const int groups = kMergeThreads / D;
  const int tid = threadIdx.x, d = tid % D, gi = tid / D;
  const int n_sh = kBeside ? a.n_shared_split : 0;
  const int n_slots = kSolo ? unit_slots(a.n_split_max, n_sh) : a.n_split_max;
  const float* ml = a.part_ml + row_head * n_slots * 2;
  const float* acc = a.part_acc + row_head * n_slots * D + d;
  const int ctx = a.ctx_lens[b];
  if (ctx < 0 || ctx > a.max_ctx_len) return;
  const int win = layer_window(a, l);
  const int lo = window_start(win, ctx + 1);
  const int n_split = split_count(ctx + 1, lo);
  const bool shared = kSolo ? kBeside : win == 0 && a.n_shared_split > 0;
  if (!kSolo && n_split == 1 && !shared) return;           // written by the split kernel
  const int n_unit = min((ctx - split_base(lo)) / kUnit + 1, 4 * n_split);   // units that hold keys (kSolo)
  if (kSolo && n_unit == 1 && !shared) return;             // written by the split kernel
  auto slot_of = [&](int s) { return kSolo ? unit_slot(s, n_sh) : s; };
  auto has_unit = [&](int s, int u) { return s >= n_sh && s * 4 + u < n_unit; };   // kSolo, u > 0
  extern __shared__ float s_mem[];
  float* s_m = s_mem;                                      // [split] reference, then weight
  float* s_l = s_m + a.n_split_max;                        // [split] sum
  float* s_u = s_l + a.n_split_max;                        // kSolo: [split][6] factors of units 1..3
  float* s_o = s_u + (kSolo ? 6 : 0) * a.n_split_max;      // [kMergeChunk][D]
  __shared__ float s_max[kMergeThreads / 64];

  float mx = -INFINITY;
  for (int s = tid; s < n_split; s += kMergeThreads) {
    float2 p = *reinterpret_cast<const float2*>(ml + slot_of(s) * 2);
    if constexpr (kSolo) {
      float2 pu[3];
#pragma unroll
      for (int u = 1; u < 4; ++u) pu[u - 1] = *reinterpret_cast<const float2*>(ml + (slot_of(s) + (has_unit(s, u) ? u : 0)) * 2);
#pragma unroll
      for (int u = 1; u < 4; ++u) {
        const bool in = has_unit(s, u);
        const float m_new = fmaxf(p.x, in ? pu[u - 1].x : p.x);
        const float f_me = merge_factor(p.x, m_new);
        const float f_o = in ? merge_factor(pu[u - 1].x, m_new) : 0.0f;
        p.y = in ? fmaf(p.y, f_me, pu[u - 1].y * f_o) : p.y;
        p.x = m_new;
        s_u[s * 6 + 2 * (u - 1)] = f_me;
        s_u[s * 6 + 2 * (u - 1) + 1] = f_o;
      }
    }
    s_m[s] = p.x;
    s_l[s] = p.y;
    mx = fmaxf(mx, p.x);
  }
#pragma unroll
  for (int x = 32; x >= 1; x >>= 1) mx = fmaxf(mx, __shfl_xor(mx, x));
  if (tid % 64 == 0) s_max[tid / 64] = mx;
  __syncthreads();
  float m = s_max[0];
#pragma unroll
  for (int w = 1; w < kMergeThreads / 64; ++w) m = fmaxf(m, s_max[w]);
  for (int s = tid; s < n_split; s += kMergeThreads) s_m[s] = merge_factor(s_m[s], m);
  __syncthreads();

  float lsum = 0.0f, o = 0.0f;
  for (int c0 = 0; c0 < n_split; c0 += kMergeChunk) {
    // splits c0 + gi, + groups, ... of this chunk, two at a time
    for (int s0 = c0 + gi; s0 < min(c0 + kMergeChunk, n_split); s0 += 2 * groups) {
      float av[2][U];
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int s = min(s0 + k * groups, n_split - 1);
          av[k][u] = acc[(int64_t)(slot_of(s) + (u > 0 && has_unit(s, u) ? u : 0)) * D];
        }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int s = s0 + k * groups;
        float v = av[k][0];
        if constexpr (kSolo) {
          const float* f = s_u + min(s, n_split - 1) * 6;
#pragma unroll
          for (int u = 1; u < 4; ++u) v = has_unit(s, u) ? fmaf(v, f[2 * (u - 1)], av[k][u] * f[2 * (u - 1) + 1]) : v;
        }
        if (s < min(c0 + kMergeChunk, n_split)) s_o[(s - c0) * D + d] = v;
      }
    }
    __syncthreads();
    if (gi == 0) {
      const int n = min(kMergeChunk, n_split - c0);
#pragma unroll 8
      for (int i = 0; i < n; ++i) {
        const float f = s_m[c0 + i];
        lsum = fmaf(s_l[c0 + i], f, lsum);
        o = fmaf(s_o[i * D + d], f, o);
      }
    }
    __syncthreads();
  }
  if (gi == 0) a.out[row_head * D + d] = o / lsum;
}

// merge_splits_kernel<false> serves rows that leave lanes idle: up to two workgroups on each of the 256 CUs.
// Above, a row's 256 lanes are enough and most of its 1,024 only wait.  16 query heads x 256, over 66 splits: 256 rows
// 10.2 us against 11.8 on 256 lanes, 512 rows 12.4 against 13.0, 1,024 rows 22.5 against 17.1, 24,576 rows 654 against 313;
// over 18 splits: 5.2 / 6.3, 6.3 / 6.6, 11.0 / 8.6.  More splits than fit its LDS combine on 256 lanes too.
constexpr int64_t kMergeRows = 512;
// Units of up to so many splits are merged on 256 lanes a row (4 layers x 8 sequences, 512 rows over one split: 17 us
// a call against 21; 768 rows over 3: 25.8 / 28.3), of more on 1,024.
constexpr int kMergeFewSplits = 4;
constexpr size_t kMergeLds = 65536 - 256;      // dynamic: its static arrays and this stay within 64 KiB
// Bytes of dynamic LDS it takes.
size_t merge_lds(const DecodeArgs& a) {
  return ((size_t)a.n_split_max * (a.solo ? 8 : 2) + (size_t)kMergeChunk * a.D) * sizeof(float);
}

template <int D>
hipError_t launch_decode_g(const DecodeArgs& a, hipStream_t stream) {
  const int64_t n_blocks = decode_items(a);
  switch (a.group) {
    case 1: decode_kernel<D, 1><<<dim3((unsigned)n_blocks), kThreads, 0, stream>>>(a); break;
    case 2: decode_kernel<D, 2><<<dim3((unsigned)n_blocks), kThreads, 0, stream>>>(a); break;
    case 4: decode_kernel<D, 4><<<dim3((unsigned)n_blocks), kThreads, 0, stream>>>(a); break;
    case 8: decode_kernel<D, 8><<<dim3((unsigned)n_blocks), kThreads, 0, stream>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_decode_f32(const DecodeArgs& a, hipStream_t stream) {
  switch (a.D) {
    case 64: return launch_decode_g<64>(a, stream);
    case 128: return launch_decode_g<128>(a, stream);
    case 256: return launch_decode_g<256>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

// Suffix prefill over shared pages: each row's two partials (the shared pages, from the
// shared-split mode of the MFMA kernel; the sequence's own keys, from its per-sequence mode)
// combined in that order, on full-attention layers.
__global__ __launch_bounds__(kThreads) void prefill_combine_kernel(const PrefillArgs a, int64_t n_rows) {
  // a workgroup per (layer, sequence, chunk row, query head), grid-strided
  for (int64_t row_head = blockIdx.x; row_head < n_rows; row_head += gridDim.x) {
    const int b = (int)((row_head / ((int64_t)a.Hq * a.chunk)) % a.batch);
    const int l = (int)(row_head / ((int64_t)a.Hq * a.chunk * a.batch));
    if (layer_window(a, l) != 0) continue;        // written by the per-sequence kernel
    const int ctx = a.ctx_lens[b];
    if (ctx < 0 || ctx > a.max_ctx_len) continue;
    const float* ml = a.part_ml + row_head * a.n_split_max * 2;
    const float* acc = a.part_acc + row_head * a.n_split_max * a.D;
    for (int d = threadIdx.x; d < a.D; d += kThreads)
      a.out[row_head * a.D + d] = combine_splits<2>(ml, acc + d, a.D, a.n_split_max);
  }
}

// Prefill of fp32 caches, and with 8 query heads per KV head: each row's partials over the kSplit-key segments (absolute
// multiples) that hold its visible keys, combined in ascending order.  One element per lane.
__global__ __launch_bounds__(kThreads) void prefill_segments_kernel(const PrefillArgs a, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
    const int64_t row_head = i / a.D;
    const int row = (int)((row_head / a.Hq) % a.chunk);
    const int b = (int)((row_head / ((int64_t)a.Hq * a.chunk)) % a.batch);
    const int l = (int)(row_head / ((int64_t)a.Hq * a.chunk * a.batch));
    const int ctx = a.ctx_lens[b];
    if (ctx < 0 || ctx > a.max_ctx_len) continue;
    const int n_keys = ctx + row + 1;
    const int s0 = window_start(layer_window(a, l), n_keys) / kSplit;
    const int64_t p0 = row_head * a.n_split_max + s0;
    a.out[i] = combine_splits(a.part_ml + p0 * 2, a.part_acc + p0 * a.D + i % a.D, a.D, (n_keys - 1) / kSplit - s0 + 1);
  }
}

}  // namespace

hipError_t launch_prefill_segments(const PrefillArgs& a, hipStream_t stream) {
  const int64_t n = (int64_t)a.n_layers * a.batch * a.chunk * a.Hq * a.D;
  const unsigned n_wg = (unsigned)std::min<int64_t>((n + kThreads - 1) / kThreads, int64_t(1) << 22);
  prefill_segments_kernel<<<dim3(n_wg), kThreads, 0, stream>>>(a, n);
  return hipGetLastError();
}

hipError_t launch_prefill_combine(const PrefillArgs& a, hipStream_t stream) {
  const int64_t n_rows = (int64_t)a.n_layers * a.batch * a.chunk * a.Hq;
  if (n_rows <= 0) return hipSuccess;
  const unsigned n_wg = (unsigned)std::min<int64_t>(n_rows, int64_t(1) << 22);   // 2^30 threads at most
  prefill_combine_kernel<<<dim3(n_wg), kThreads, 0, stream>>>(a, n_rows);
  return hipGetLastError();
}

hipError_t launch_decode(const DecodeArgs& a, int dtype, hipStream_t stream) {
  const hipError_t e = decode_items(a) == 0   ? hipSuccess
                       : dtype == kDtypeF32 ? launch_decode_f32(a, stream)
                                            : launch_decode_mfma(a, dtype, stream);
  if (e != hipSuccess) return e;
  if (a.n_split_max == 1 && a.n_shared_split == 0 && !a.solo) return hipSuccess;   // every row is written
  const int64_t n_rows = (int64_t)a.n_layers * a.batch * a.Hq;
  const dim3 grid((unsigned)n_rows);
  if (a.solo && a.n_shared_split > 0)
    merge_splits_kernel<true, 1024, true><<<grid, 1024, merge_lds(a), stream>>>(a);
  else if (a.solo && a.n_split_max <= kMergeFewSplits)
    merge_splits_kernel<true, 256><<<grid, 256, merge_lds(a), stream>>>(a);
  else if (a.solo)
    merge_splits_kernel<true, 1024><<<grid, 1024, merge_lds(a), stream>>>(a);
  else if (a.n_split_max > 16 && merge_lds(a) <= kMergeLds && n_rows <= kMergeRows)
    merge_splits_kernel<false, 1024><<<grid, 1024, merge_lds(a), stream>>>(a);
  else
    decode_merge_kernel<<<grid, kThreads, 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace kvg
