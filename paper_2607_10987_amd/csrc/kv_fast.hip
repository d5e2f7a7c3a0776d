// MFMA append path (bf16, head_dim 128).
#include "kv_fast.h"

namespace kvs {

bool decode_mfma_ok(const PoolGeom& g, int dtype, const AppendDesc& a);
void decode_scratch(const PoolGeom& g, const AppendDesc& a, bool wide, size_t* per_layer,
                    size_t* fixed);
size_t decode_scratch_bound(const PoolGeom& g, int dtype, int64_t tokens, int64_t batch,
                            int64_t max_keys);
void decode_query(const PoolGeom& g, const AppendDesc& a, bool wide, int64_t* out);
hipError_t launch_decode_attn(const PoolGeom& g, const void* qbuf, const AppendDesc& a, bool wide,
                              void* part, void* plan, int lc, int l0, hipStream_t s);
hipError_t launch_decode_merge(const PoolGeom& g, const AppendDesc& a, bool wide, void* o,
                               const void* part, const void* plan, int l0, int lc,
                               hipStream_t s);

bool attn_packed_ok(const PoolGeom& g, int dtype, const AppendDesc& a);
size_t attn_packed_bytes(const PoolGeom& g, const AppendDesc& a);
hipError_t launch_attn_packed(const PoolGeom& g, const void* qbuf, const AppendDesc& a, void* o,
                              void* plan, int l0, int lc, hipStream_t s);

namespace {
// The split-key kernels: every T = 1 call, T > 1 calls in the wide form.
bool takes_decode(const PoolGeom& g, int dtype, const AppendDesc& a, AttnForm form) {
  return (a.T == 1 || form == kWide) && decode_mfma_ok(g, dtype, a);
}
}  // namespace

bool fast_wide_ok(const PoolGeom& g, int dtype, const AppendDesc& a) {
  return decode_mfma_ok(g, dtype, a) || attn_packed_ok(g, dtype, a);
}

void fast_scratch_need(const PoolGeom& g, int dtype, const AppendDesc& a, AttnForm form,
                       size_t* per_layer, size_t* fixed) {
  *per_layer = *fixed = 0;
  if (takes_decode(g, dtype, a, form))
    decode_scratch(g, a, form == kWide, per_layer, fixed);
  else if (form == kWide && attn_packed_ok(g, dtype, a))
    *fixed = attn_packed_bytes(g, a);
}

size_t fast_scratch_bound(const PoolGeom& g, int dtype, int64_t tokens, int32_t batch,
                          int64_t max_keys) {
  // split-key partials and the work-unit plan (more than a packed call's counts)
  return decode_scratch_bound(g, dtype, tokens, batch, max_keys);
}

hipError_t launch_qkv_mfma(const PoolGeom& g, const void* x, const void* w, int64_t w_stride,
                           const AppendDesc& a, void* qbuf, int l0, int lc, hipStream_t s);

hipError_t launch_qkv_fast(const PoolGeom& g, int dtype, const void* x, const void* w,
                           int64_t w_stride, const AppendDesc& a, void* qbuf, int l0, int lc,
                           hipStream_t s, bool* done) {
  *done = false;
  if (!qkv_mfma_ok(g, dtype)) return hipSuccess;
  *done = true;
  return launch_qkv_mfma(g, x, w, w_stride, a, qbuf, l0, lc, s);
}

bool attn_mfma_ok(const PoolGeom& g, int dtype, const AppendDesc& a);
hipError_t launch_attn_prefill(const PoolGeom& g, const void* qbuf, const AppendDesc& a, void* o,
                               int l0, int lc, hipStream_t s);

AttnPath fast_attn_query(const PoolGeom& g, int dtype, const AppendDesc& a, AttnForm form,
                         int64_t* out) {
  if (takes_decode(g, dtype, a, form)) {
    decode_query(g, a, form == kWide, out);
    return kPathSplitKey;
  }
  if (!attn_mfma_ok(g, dtype, a)) return kPathPortable;
  return form == kWide && attn_packed_ok(g, dtype, a) ? kPathPacked : kPathPrefill;
}

hipError_t launch_attn_fast(const PoolGeom& g, int dtype, const void* qbuf, const AppendDesc& a,
                            AttnForm form, void* o, void* part, void* plan, int l0, int lc,
                            hipStream_t s, bool* done, bool* merge) {
  *done = false;
  *merge = false;
  if (takes_decode(g, dtype, a, form)) {
    *done = true;
    *merge = true;
    return launch_decode_attn(g, qbuf, a, form == kWide, part, plan, lc, l0, s);
  }
  if (!attn_mfma_ok(g, dtype, a)) return hipSuccess;
  *done = true;
  if (form == kWide && attn_packed_ok(g, dtype, a))
    return launch_attn_packed(g, qbuf, a, o, plan, l0, lc, s);
  return launch_attn_prefill(g, qbuf, a, o, l0, lc, s);
}

hipError_t launch_attn_merge(const PoolGeom& g, int, const AppendDesc& a, AttnForm form, void* o,
                             const void* part, const void* plan, int l0, int lc, hipStream_t s) {
  return launch_decode_merge(g, a, form == kWide, o, part, plan, l0, lc, s);
}

}  // namespace kvs
