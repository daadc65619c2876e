// Host-side launchers of the libkvg kernels (implemented next to each kernel).
#pragma once

#include <hip/hip_runtime.h>

#include "kvg.h"
#include "kvg_device.h"

namespace kvg {

// A launch of `wgs` workgroups of `threads` threads fits the dispatch limits (grid size in
// threads below 2^32).
inline bool fits_grid(int64_t wgs, int threads) { return wgs >= 0 && wgs * (int64_t)threads <= (int64_t)UINT32_MAX; }

// `dtype` is the cache's storage dtype code (kDtypeF32, kDtypeBf16, kDtypeFp8).
hipError_t launch_append(const AppendArgs& a, int dtype, hipStream_t stream);
hipError_t launch_deposit(const CopyArgs& a, hipStream_t stream);
hipError_t launch_graft(const CopyArgs& a, int dtype, hipStream_t stream);
// workgroups (256 threads each) of the deposit's and of the graft's launch (own position or
// relocated), for the host's launch-size checks
int64_t copy_workgroups(const CopyArgs& a, int dtype);
// the prefill of an fp32 cache (kvg_prefill_f32.hip): a.q holds fp32 queries, a.n_qt 32-pair tiles,
// a.n_split_max kSplit-key splits.  Partials (a.part_acc) where there are several splits, or, with a workgroup per
// unit (kF32Units a split), several units
constexpr int kF32Units = 4;
enum class F32Form {
  kSplits,    // a workgroup per split
  kUnits,     // a workgroup per unit
  kNarrow,    // a workgroup per unit and a few (row, query head) pairs, on the vector ALUs
};
hipError_t launch_prefill_f32(const PrefillArgs& a, F32Form form, hipStream_t stream);
inline int64_t prefill_f32_workgroups(const PrefillArgs& a) {
  return (int64_t)a.n_layers * a.batch * a.Hkv * a.n_split_max * a.n_qt;
}
hipError_t launch_prefill_mfma(const PrefillArgs& a, int dtype, hipStream_t stream);
// waves (32 query rows each) per workgroup of the MFMA prefill at head_dim D; a workgroup
// covers 32 * waves / group rows of each of the group's query heads
int prefill_mfma_waves(int D);
// workgroups that share the query heads of one KV head (more than one where a workgroup has
// fewer waves than the KV head has query heads)
int prefill_head_sets(int D, int group);
// decode partials of splits [0, a.n_shared_split) of every full-attention layer, for a batch
// whose sequences share those pages; a.q holds the rotated queries [n_layers][batch][Hq][D]
hipError_t launch_shared_splits(const PrefillArgs& a, int dtype, hipStream_t stream);
// a suffix prefill over shared pages: out = the rows' n_split_max partials combined in order
hipError_t launch_prefill_combine(const PrefillArgs& a, hipStream_t stream);
// fp32 caches, and 8 query heads per KV head: out = each row's partials of the kSplit-key segments it
// sees
hipError_t launch_prefill_segments(const PrefillArgs& a, hipStream_t stream);
hipError_t launch_decode(const DecodeArgs& a, int dtype, hipStream_t stream);
// work items (a split of a KV head of a layer of a sequence) of a decode's grid
inline int64_t decode_items(const DecodeArgs& a) {
  return (int64_t)a.batch * a.Hkv * ((int64_t)a.n_full * a.n_split_full + (int64_t)(a.n_layers - a.n_full) * a.n_split_win);
}
// its split kernel for bf16 and fp8 caches (kvg_decode_mfma.hip); K and V bytes of one of its stages, for cache
// rows of RB bytes
constexpr int kLdsBytes = 160 << 10;       // of a CU
constexpr int decode_stage_bytes(int RB) { return RB >= 256 ? 16384 : 8192; }
hipError_t launch_decode_mfma(const DecodeArgs& a, int dtype, hipStream_t stream);


// The decode call split at its workspace (kvg_api.cpp): argument validation, the workspace
// size, and the launches on a given workspace (which is checked against the size).
int decode_attn_check(const kvg_cache* cache, const kvg_seqs* seqs, const kvg_rope* rope, int32_t layer0,
                      int32_t n_layers, const void* q_raw, const void* k_raw, const void* v_raw, float scale,
                      float* out);
size_t decode_attn_ws_bytes(const kvg_cache* cache, const kvg_seqs* seqs, int32_t n_layers);
int decode_attn_launch(const kvg_cache* cache, const kvg_seqs* seqs, const kvg_rope* rope, int32_t layer0,
                       int32_t n_layers, const void* q_raw, const void* k_raw, const void* v_raw, float scale,
                       float* out, void* ws, size_t ws_bytes, hipStream_t stream);

}  // namespace kvg
