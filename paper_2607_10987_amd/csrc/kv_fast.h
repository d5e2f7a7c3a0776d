// MFMA (bf16) append path: projection GEMM with fused RoPE and paged store,
// causal prefill attention, and split-K decode attention.  Each launcher sets
// *done = false (and enqueues nothing) when the shape is not covered, in which
// case the portable kernels of kv_generic.hip run instead.
#pragma once

#include "kv_internal.h"

namespace kvs {

// Which attention a call takes beyond the Q buffer's needs.  kPlain asks for
// the least scratch (prefill attention for T > 1, the smallest split-key
// layout for T = 1); kWide is the split-key form that follows divergences
// inside a chunk, or for more query vectors the packed prefill attention,
// taken when its scratch does not cost the call layers per group.  kWide is
// not offered for every call.
enum AttnForm { kPlain = 0, kWide = 1 };
bool fast_wide_ok(const PoolGeom& g, int dtype, const AppendDesc& a);
// Scratch bytes the fast attention needs beyond the Q buffer for this call:
// *per_layer for each layer of a group in flight (split-key partials) and
// *fixed once per call (the decode work plan), both multiples of 256.
void fast_scratch_need(const PoolGeom& g, int dtype, const AppendDesc& a, AttnForm form,
                       size_t* per_layer, size_t* fixed);
// An upper bound of the same for calls of `tokens` new tokens over at most
// `max_keys` keys per state.
size_t fast_scratch_bound(const PoolGeom& g, int dtype, int64_t tokens, int32_t batch,
                          int64_t max_keys);

// The bf16 projection of M token rows and lc layers on a device of n_cu CUs:
// its kernel, token rows per tile and stages of the weights (kTiles).
struct QkvPick {
  enum Kernel { kStream, kRowsLds, kRows, kTile32, kTiles } kernel;
  int rows, stages;
};
bool qkv_mfma_ok(const PoolGeom& g, int dtype);
QkvPick pick_qkv(const PoolGeom& g, int M, int lc, int n_cu);

// How a call's attention runs in this form (for tests): its path, and for the
// split-key path keys per chunk, chunks, lists and the plan kernel's dynamic LDS
// bytes in out[0..3].
enum AttnPath { kPathPortable = 0, kPathPrefill, kPathPacked, kPathSplitKey };
AttnPath fast_attn_query(const PoolGeom& g, int dtype, const AppendDesc& a, AttnForm form,
                         int64_t* out);

hipError_t launch_qkv_fast(const PoolGeom& g, int dtype, const void* x, const void* w,
                           int64_t w_stride, const AppendDesc& a, void* qbuf, int l0, int lc,
                           hipStream_t s, bool* done);
// part: per_layer bytes for each layer of the group; plan: the fixed bytes,
// written by the group that starts at layer 0 and read by every group.
// *merge = true when the launch wrote split-key partials that
// launch_attn_merge must combine into o.
hipError_t launch_attn_fast(const PoolGeom& g, int dtype, const void* qbuf, const AppendDesc& a,
                            AttnForm form, void* o, void* part, void* plan, int l0, int lc,
                            hipStream_t s, bool* done, bool* merge);
hipError_t launch_attn_merge(const PoolGeom& g, int dtype, const AppendDesc& a, AttnForm form,
                             void* o, const void* part, const void* plan, int l0, int lc,
                             hipStream_t s);

}  // namespace kvs
