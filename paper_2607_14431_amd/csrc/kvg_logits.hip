// Synthetic logit head over hidden vectors, and the comparison of two logit sets.
//
// The exactness verdict is taken on logits: SHA-256 equality of their bytes (Eq. 1), and as
// corollaries a zero KL divergence between the two softmax distributions and equal argmax
// (Eq. 2); the model's logits pass through a soft cap (Sec. 4.2).  The head here is
//   logits[r][v] = cap * tanh(z / cap),  z = sum_k bf16(hidden[r][k]) * W[v][k]
// (z itself when cap = 0), fp32 accumulation, W bf16 [V][H].
//
// Head kernel: the contraction runs on v_mfma_f32_32x32x16_bf16 with A = 32 vocabulary rows
// of W and B = 32 hidden rows, so a decode batch of up to 32 rows reads W exactly once; W
// streams from HBM and bounds the kernel.  Both operands are in the fragment-major packing
// (kvg_logits.h): W packed once by kvg_logits_pack, the hidden rows converted to bf16 and
// packed into the workspace by each call.  Lane (r, h) of fragment t of 64-element block kb
// holds row r and elements 64 kb + 32 h + 8 t .. + 8, for both operands, so the MFMA sums
// every element of the block exactly once, and each fragment load of a wave is 1 KiB of
// consecutive bytes: a wave streams each of its four 32-row blocks of W as one sequential
// run of H * 64 bytes.  A wave owns 128 vocabulary rows (four accumulators sharing each B
// fragment) and keeps two blocks in flight.  Hidden rows past the input are zero; vocabulary
// blocks past the padded end re-read the last block and are not stored.
//
// Compare kernel: one workgroup per row: first-index argmax of each logit vector, the log-sum-
// exp of each and KL(softmax(a) || softmax(b)) = sum_i p_i ((a_i - b_i) - (lse_a - lse_b)),
// in fp64 with fixed-order reductions, so byte-equal inputs give exactly 0.
#include "kvg_logits.h"

#include <math.h>

#include <algorithm>

namespace kvg {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x8 __attribute__((ext_vector_type(8)));

constexpr int kThreads = 256;

__device__ __forceinline__ uint4 ld16(const uint16_t* p) { return *reinterpret_cast<const uint4*>(p); }
// W is streamed once per launch (nontemporal loads): one row 372 -> 337 us, 50 rows
// 448 -> 428 us at 262,144 x 4,096.
typedef unsigned int u32x4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld16_stream(const uint16_t* p) {
  const u32x4v v = __builtin_nontemporal_load(reinterpret_cast<const u32x4v*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ bf16x8 as_bf16x8(const uint4& v) { return __builtin_bit_cast(bf16x8, v); }

// Position of packed 16-byte unit u: matrix row and first element (see packed_unit).
struct UnitPos {
  int64_t row, k;
};
__device__ __forceinline__ UnitPos unit_pos(int64_t u, int n_kb) {
  const int lane = (int)(u & 63);
  const int t = (int)((u >> 6) & 3);
  const int m = (int)((u >> 8) & 3);
  const int64_t rest = u >> 10;
  const int64_t kb = rest % n_kb, blk = rest / n_kb;
  return {kPackRows * blk + 32 * m + (lane & 31), 64 * kb + 32 * (lane >> 5) + 8 * t};
}

// hidden fp32 [rows][H] -> packed bf16, nearest-even; padding rows are zero
__global__ __launch_bounds__(kThreads) void hidden_pack_kernel(const LogitArgs a) {
  const int64_t u = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (u >= (int64_t)a.rows_pad * a.H / 8) return;
  const UnitPos p = unit_pos(u, a.H / 64);
  uint4 o = make_uint4(0, 0, 0, 0);
  if (p.row < a.rows) {
    const float* src = a.hidden + p.row * a.H + p.k;
    const float4 x0 = *reinterpret_cast<const float4*>(src);
    const float4 x1 = *reinterpret_cast<const float4*>(src + 4);
    const f32x8 x = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
    o = __builtin_bit_cast(uint4, __builtin_convertvector(x, bf16x8));
  }
  *reinterpret_cast<uint4*>(a.hidden_packed + u * 8) = o;
}

// W bf16 [V][H] row-major -> packed; rows past V are zero
__global__ __launch_bounds__(kThreads) void weight_pack_kernel(const PackArgs a) {
  const int64_t u = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (u >= packed_rows(a.V) * a.H / 8) return;
  const UnitPos p = unit_pos(u, a.H / 64);
  const uint4 o = p.row < a.V ? ld16(a.w + p.row * a.H + p.k) : make_uint4(0, 0, 0, 0);
  *reinterpret_cast<uint4*>(a.packed + u * 8) = o;
}

// A wave owns MB 32-row blocks of the vocabulary and NB 32-row tiles of hidden rows: MB x NB
// = 4 accumulators.  MB = 4, NB = 1 serves up to 32 hidden rows (a decode batch) with one
// read of W; MB = 2, NB = 2 and MB = 1, NB = 4 serve up to 64 and 128 rows per read.
template <int MB, int NB>
struct Frags {
  uint4 w[MB][4];    // [vocab block][fragment]
  uint4 h[NB][4];    // [row tile][fragment]
};

template <int MB, int NB>
__global__ __launch_bounds__(kThreads) void logit_head_kernel(const LogitArgs a) {
  constexpr int kWaveVocab = 32 * MB;
  constexpr int kGroupVocab = 4 * kWaveVocab;
  constexpr int kRows = 32 * NB;
  const int n_vt = (a.V + kGroupVocab - 1) / kGroupVocab;
  const int vt = blockIdx.x % n_vt;
  const int nt = blockIdx.x / n_vt;              // group of kRows hidden rows
  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  const int lr = lane & 31, lh = lane >> 5;
  const int v0 = vt * kGroupVocab + wave * kWaveVocab;
  if (v0 >= a.V) return;                         // no barrier below: a whole wave may leave
  const int r0 = nt * kRows;

  const int nk = a.H / 64;
  const int last_b32 = (int)(packed_rows(a.V) / 32) - 1;   // padded blocks hold zeros
  const uint16_t* wblk[MB];
  const uint16_t* hblk[NB];
#pragma unroll
  for (int m = 0; m < MB; ++m) wblk[m] = a.w_packed + packed_unit(min(v0 / 32 + m, last_b32), 0, 0, lane, nk) * 8;
#pragma unroll
  for (int n = 0; n < NB; ++n) hblk[n] = a.hidden_packed + packed_unit(r0 / 32 + n, 0, 0, lane, nk) * 8;

  // step kb of a 128-row block starts 16 units of 64 lanes (16 KiB) after step kb - 1
  auto load = [&](int kb, Frags<MB, NB>& f) {
    const int64_t off = (int64_t)kb * 16 * 64 * 8;
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int t = 0; t < 4; ++t) f.w[m][t] = ld16_stream(wblk[m] + off + t * 64 * 8);
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int t = 0; t < 4; ++t) f.h[n][t] = ld16(hblk[n] + off + t * 64 * 8);
  };
  f32x16 acc[MB][NB];
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[m][n][q] = 0.0f;
  auto compute = [&](const Frags<MB, NB>& f) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n)
          acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(f.w[m][t]), as_bf16x8(f.h[n][t]),
                                                              acc[m][n], 0, 0, 0);
  };

  // H is a multiple of 128, so steps come in pairs; every load is unconditional (the last
  // one re-reads the final step), which keeps the next step's loads in flight across the
  // loop's back edge.  The scheduling barriers keep each step's loads where they are
  // issued here (the scheduler would otherwise sink them towards their use).
  Frags<MB, NB> x, y;
  load(0, x);
  for (int kb = 0; kb < nk; kb += 2) {
    load(kb + 1, y);
    __builtin_amdgcn_sched_barrier(0);
    compute(x);
    __builtin_amdgcn_sched_barrier(0);
    load(min(kb + 2, nk - 1), x);
    __builtin_amdgcn_sched_barrier(0);
    compute(y);
    __builtin_amdgcn_sched_barrier(0);
  }

  // lane (r, h) holds, in accumulator element q of (m, n), hidden row r0 + 32 n + r and
  // vocabulary row v0 + 32 m + 8 (q / 4) + 4 h + q % 4
  const bool vec = (a.V & 3) == 0;
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const int row = r0 + 32 * n + lr;
    if (row >= a.rows) continue;
    float* orow = a.out + (int64_t)row * a.V;
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int v = v0 + 32 * m + 8 * q4 + 4 * lh;
        float l[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float z = acc[m][n][4 * q4 + e];
          l[e] = a.cap > 0.0f ? a.cap * tanhf(z / a.cap) : z;
        }
        if (vec && v + 3 < a.V) {
          *reinterpret_cast<float4*>(orow + v) = make_float4(l[0], l[1], l[2], l[3]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (v + e < a.V) orow[v + e] = l[e];
        }
      }
  }
}

// ---------------------------------------------------------------------------- comparison
// One workgroup per row at most (the call has no workspace to combine more in), so a long row is bound by
// what one CU reads and exponentiates.  One pass over both rows: with a reference r the running sums
//   A = sum e^(a - r_a),  T = sum e^(a - r_a) (a - b),  B = sum e^(b - r_b)
// give lse_a = r_a + log A, lse_b = r_b + log B and KL = T / A - (lse_a - lse_b), two
// exponentials an element.  fp64's range lets a lane keep its first value as the reference until
// one exceeds it by e^300.  50 rows of 262,144: 141 us; three passes (maximum, sums, KL) of
// 256 lanes with the library's exp: 1,108 us.
constexpr double kRaise = 300.0;

struct ArgMax {
  float v;
  int i;
};

// the larger value; of equal values the smaller index (the first maximum)
__device__ __forceinline__ ArgMax better(ArgMax x, ArgMax y) {
  return (y.v > x.v || (y.v == x.v && y.i < x.i)) ? y : x;
}

// e^x for x <= kRaise, in fp64: x = (64 k + j) ln2 / 64 + r, |r| <= ln2 / 128, so
// e^x = 2^k 2^(j/64) e^r with the table tab[j] = 2^(j/64) and e^r - 1 by its series to r^5
// (the rest is below 4e-17).  Below the smallest subnormal the result is an exact 0, so that a
// logit of -inf weighs what it should.
__device__ __forceinline__ double exp_table(double x, const double* tab) {
  constexpr double kInv = 92.332482616893656877;               // 64 / ln 2
  constexpr double kHi = 0x1.62e42fefa39efp-7, kLo = 0x1.abc9e3b39803fp-62;   // ln 2 / 64
  const double xc = x >= -750.0 ? x : -750.0;      // NaN too: the conversion needs a number
  const double n = __builtin_rint(xc * kInv);
  const double r = fma(-n, kLo, fma(-n, kHi, xc));
  const int m = (int)n;
  const double p = fma(r * r, fma(r, fma(r, fma(r, 1.0 / 120.0, 1.0 / 24.0), 1.0 / 6.0), 0.5), r);
  const double t = tab[m & 63];
  const double y = __builtin_ldexp(fma(t, p, t), m >> 6);
  return x >= -750.0 ? y : x < -750.0 ? 0.0 : x;
}

struct RowSums {
  double ra, rb, sa, sb, t;      // references, sums, weighted differences
  ArgMax ma, mb;
};

__device__ __forceinline__ void add_element(RowSums& s, float af, float bf, int i, const double* tab) {
  s.ma = better(s.ma, ArgMax{af, i});
  s.mb = better(s.mb, ArgMax{bf, i});
  const double a = af, b = bf;
  if (__builtin_amdgcn_ballot_w64(a - s.ra > kRaise || b - s.rb > kRaise) != 0) {   // rare
    if (a - s.ra > kRaise) {
      const double f = exp_table(s.ra - a, tab);
      s.sa *= f;
      s.t *= f;
      s.ra = a;
    }
    if (b - s.rb > kRaise) {
      s.sb *= exp_table(s.rb - b, tab);
      s.rb = b;
    }
  }
  const double ea = exp_table(a - s.ra, tab);
  s.sa += ea;
  s.t = fma(ea, a - b, s.t);
  s.sb += exp_table(b - s.rb, tab);
}

struct Refs {
  double a, b;
};
struct Sums {
  double a, b, t;
  ArgMax ma, mb;
};
__device__ __forceinline__ Refs shuffle(const Refs& x, int m) { return {__shfl_xor(x.a, m), __shfl_xor(x.b, m)}; }
__device__ __forceinline__ Sums shuffle(const Sums& x, int m) {
  return {__shfl_xor(x.a, m), __shfl_xor(x.b, m), __shfl_xor(x.t, m), {__shfl_xor(x.ma.v, m), __shfl_xor(x.ma.i, m)},
          {__shfl_xor(x.mb.v, m), __shfl_xor(x.mb.i, m)}};
}

// x combined with y over the row's lanes: over a wave by shuffles, over several waves in their order
template <int kLanes, typename X, typename Op>
__device__ __forceinline__ X over_row(X x, Op op, X* sh) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) x = op(x, shuffle(x, m));
  if constexpr (kLanes > 64) {
    if (threadIdx.x % 64 == 0) sh[threadIdx.x / 64] = x;
    __syncthreads();
    x = sh[0];
#pragma unroll
    for (int w = 1; w < kLanes / 64; ++w) x = op(x, sh[w]);
  }
  return x;
}

// kVec: rows of 16-byte vectors (V a multiple of 4 and both buffers aligned).  kLanes: of a row.
template <bool kVec, int kLanes>
__global__ __launch_bounds__(kLanes < kThreads ? kThreads : kLanes, 8) void logit_compare_kernel(const CompareArgs c) {
  constexpr int kRowsPer = kLanes < kThreads ? kThreads / kLanes : 1;
  __shared__ double tab[64];
  __shared__ Refs sh_refs[kLanes / 64];
  __shared__ Sums sh_sums[kLanes / 64];
  const int tid = threadIdx.x % kLanes;
  const int row = blockIdx.x * kRowsPer + threadIdx.x / kLanes;
  if (threadIdx.x < 64) tab[threadIdx.x] = exp2(threadIdx.x / 64.0);
  __syncthreads();
  if (row >= c.rows) return;                       // whole waves (kLanes 64)
  const float* a = c.a + (int64_t)row * c.V;
  const float* b = c.b + (int64_t)row * c.V;

  // a reference far below every finite logit stands for "none yet" (it is raised at the first)
  RowSums s{-1e300, -1e300, 0.0, 0.0, 0.0, {-INFINITY, c.V}, {-INFINITY, c.V}};
  if constexpr (kVec) {
    const int n4 = c.V / 4;
    const float4* a4 = reinterpret_cast<const float4*>(a);
    const float4* b4 = reinterpret_cast<const float4*>(b);
    // the next vectors are requested before the current ones are used (the last lanes' re-read
    // their own)
    float4 na = a4[min(tid, n4 - 1)], nb = b4[min(tid, n4 - 1)];
    for (int i = tid; i < n4; i += kLanes) {
      const float4 x = na, y = nb;
      const int next = min(i + kLanes, n4 - 1);
      na = a4[next];
      nb = b4[next];
      add_element(s, x.x, y.x, 4 * i, tab);
      add_element(s, x.y, y.y, 4 * i + 1, tab);
      add_element(s, x.z, y.z, 4 * i + 2, tab);
      add_element(s, x.w, y.w, 4 * i + 3, tab);
    }
  } else {
    for (int i = tid; i < c.V; i += kLanes) add_element(s, a[i], b[i], i, tab);
  }

  // every lane's sums over the row's largest references, then added in a fixed tree
  const Refs r = over_row<kLanes>(
      Refs{s.ra, s.rb}, [](const Refs& x, const Refs& y) { return Refs{fmax(x.a, y.a), fmax(x.b, y.b)}; }, sh_refs);
  const double fa = exp_table(s.ra - r.a, tab);
  const Sums sum = over_row<kLanes>(
      Sums{s.sa * fa, s.sb * exp_table(s.rb - r.b, tab), s.t * fa, s.ma, s.mb},
      [](const Sums& x, const Sums& y) {
        return Sums{x.a + y.a, x.b + y.b, x.t + y.t, better(x.ma, y.ma), better(x.mb, y.mb)};
      },
      sh_sums);
  if (tid == 0) {
    const double lse_a = r.a + log(sum.a), lse_b = r.b + log(sum.b);
    c.kl[row] = sum.t / sum.a - (lse_a - lse_b);
    c.arg_a[row] = sum.ma.i;
    c.arg_b[row] = sum.mb.i;
  }
}

}  // namespace

template <int MB, int NB>
void launch_head(const LogitArgs& a, hipStream_t stream) {
  const int64_t n_vt = (a.V + 128 * MB - 1) / (128 * MB);
  const int64_t n_nt = (a.rows + 32 * NB - 1) / (32 * NB);
  logit_head_kernel<MB, NB><<<dim3((unsigned)(n_vt * n_nt)), kThreads, 0, stream>>>(a);
}

hipError_t launch_logits(const LogitArgs& a, hipStream_t stream) {
  const int64_t n8 = (int64_t)a.rows_pad * a.H / 8;
  hidden_pack_kernel<<<dim3((unsigned)((n8 + kThreads - 1) / kThreads)), kThreads, 0, stream>>>(a);
  if (a.rows <= 32)
    launch_head<4, 1>(a, stream);
  else if (a.rows <= 64)
    launch_head<2, 2>(a, stream);
  else
    launch_head<1, 4>(a, stream);
  return hipGetLastError();
}

hipError_t launch_logits_pack(const PackArgs& a, hipStream_t stream) {
  const int64_t n8 = packed_rows(a.V) * a.H / 8;
  weight_pack_kernel<<<dim3((unsigned)((n8 + kThreads - 1) / kThreads)), kThreads, 0, stream>>>(a);
  return hipGetLastError();
}

// Lanes of a row, by its length alone (a row's bytes do not depend on the others): what a lane does beside its
// elements (references, factors, sums over the lanes) is 2 us of a wave's time and 5 of 16 waves'.
//   us, 64 / 256 / 1024 lanes   1 row               1,000 rows             10,000 rows
//   V 100                       5.1 / 5.0 / 7.6     5.6 / 7.5 / 24.7       17 / 44 / 211
//   V 512                       5.2 / 5.1 / 7.6     6.3 / 7.8 / 24.9       22 / 45 / 216
//   V 2,048                     9.3 / 5.6 / 8.2     12 / 11 / 29           54 / 66 / 256
//   V 8,192                     29 / 10 / 12        35 / 26 / 43           196 / 207 / 399
//   V 16,384                    54 / 17 / 16        63 / 45 / 60           374 / 382 / 569
// 256 lanes in three passes: 7.9, 8.0 and 37 at V 100; 39, 96 and 748 at V 16,384.
template <bool kVec>
void launch_compare(const CompareArgs& c, hipStream_t stream) {
  if (c.V <= 512)
    logit_compare_kernel<kVec, 64><<<dim3((unsigned)((c.rows + 3) / 4)), kThreads, 0, stream>>>(c);
  else if (c.V <= 12288)
    logit_compare_kernel<kVec, 256><<<dim3((unsigned)c.rows), kThreads, 0, stream>>>(c);
  else
    logit_compare_kernel<kVec, 1024><<<dim3((unsigned)c.rows), 1024, 0, stream>>>(c);
}

hipError_t launch_logit_compare(const CompareArgs& call, hipStream_t stream) {
  constexpr int32_t kRows = 1 << 20;             // of a launch: 2^30 threads
  const bool vec = call.V % 4 == 0 && reinterpret_cast<uintptr_t>(call.a) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(call.b) % 16 == 0;
  CompareArgs c = call;
  for (int32_t row = 0; row < call.rows; row += kRows) {
    c.rows = std::min(call.rows - row, kRows);
    if (vec)
      launch_compare<true>(c, stream);
    else
      launch_compare<false>(c, stream);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    c.a += (int64_t)kRows * c.V;
    c.b += (int64_t)kRows * c.V;
    c.kl += kRows;
    c.arg_a += kRows;
    c.arg_b += kRows;
  }
  return hipSuccess;
}

}  // namespace kvg
