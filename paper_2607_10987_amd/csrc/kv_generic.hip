// Portable append path for any head_dim <= 256 (multiple of 16) and both
// storage types, in fp32 throughout: the products run on the fp32 matrix cores
// (v_mfma_f32_16x16x4_f32: fp32 operands and accumulation).  This is the path
// of float32 pools and of shapes the bf16 MFMA kernels do not cover.
//
//  k_qkv_generic: one workgroup computes 16 rotation pairs of one head (pairs
//    (i, i + dh/2), angles from the float table built in double on the host)
//    for 16 or 64 token rows of one layer, its wavefronts taking every eighth
//    16 of the contraction, and stores Q into the scratch buffer and K/V into
//    the row's paged block: block = table[slot][(n_before + t) / B], slot =
//    (n_before + t) % B.
//  k_attn_generic: one workgroup per 16 query vectors (token, head) of one KV
//    head, sequence and layer; its wavefronts take every NW-th tile of 16
//    visible keys (key index <= n_before + t) with an online (running max /
//    running sum) softmax and are combined through LDS.
//
// Both are latency-bound on the small calls they serve, so the contraction and
// the keys are split over the wavefronts of a workgroup and the operands go
// straight to registers.  A 256-token context, two 32-token appends and 8
// decode steps (d_model 256, 4 / 2 heads of 64, one layer): projections 1575
// -> 68 us, attention 1006 -> 123 us in all, against one workgroup per 32
// rows x head staged through LDS and one wavefront per (row, head).
#include <algorithm>
#include <type_traits>

#include "kv_internal.h"

namespace kvs {

namespace {

template <typename T>
__device__ inline float ld(const T* p);
template <>
__device__ inline float ld<float>(const float* p) { return *p; }
template <>
__device__ inline float ld<uint16_t>(const uint16_t* p) {
  return __uint_as_float((uint32_t)(*p) << 16);
}

template <typename T>
__device__ inline T cvt(float f);
template <>
__device__ inline float cvt<float>(float f) { return f; }
template <>
__device__ inline uint16_t cvt<uint16_t>(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

typedef float floatx4 __attribute__((ext_vector_type(4)));

// Four consecutive elements; VEC: 4-element aligned, else element-wise up to n.
template <bool VEC>
__device__ inline floatx4 ld4(const float* p, int n) {
  if (VEC) return *(const floatx4*)p;
  floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (j < n) v[j] = p[j];
  return v;
}
template <bool VEC>
__device__ inline floatx4 ld4(const uint16_t* p, int n) {
  floatx4 v = {0.f, 0.f, 0.f, 0.f};
  if (VEC) {
    const uint2 u = *(const uint2*)p;
    v[0] = __uint_as_float(u.x << 16);
    v[1] = __uint_as_float(u.x & 0xffff0000u);
    v[2] = __uint_as_float(u.y << 16);
    v[3] = __uint_as_float(u.y & 0xffff0000u);
    return v;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (j < n) v[j] = ld<uint16_t>(p + j);
  return v;
}
__device__ inline void st4(float* p, const float* v) {
  *(float4*)p = make_float4(v[0], v[1], v[2], v[3]);
}
__device__ inline void st4(uint16_t* p, const float* v) {
  *(uint2*)p = make_uint2((uint32_t)cvt<uint16_t>(v[0]) | ((uint32_t)cvt<uint16_t>(v[1]) << 16),
                          (uint32_t)cvt<uint16_t>(v[2]) | ((uint32_t)cvt<uint16_t>(v[3]) << 16));
}

constexpr int kGenWaves = 8;

// grid ((Hq + 2 Hkv) x pair tiles, token tiles, lc), block 64 kGenWaves; TJ
// token tiles of 16.  In v_mfma_f32_16x16x4_f32 lane l holds row (column) l %
// 16 at k = l / 16; with 16 contraction indices per 16-byte load, lane l takes
// 4 (l / 16) .. + 3 of both operands and feeds them to four products.
template <typename T, int TJ, bool VEC>
__global__ void __launch_bounds__(64 * kGenWaves)
k_qkv_generic(PoolGeom g, const T* __restrict__ x, const T* __restrict__ w, int64_t w_stride,
              AppendDesc a, T* __restrict__ qbuf, int l0) {
  __shared__ floatx4 red[kGenWaves][2][TJ][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int dh = g.dh, d = g.d, half = dh / 2, pt = (half + 15) / 16;
  const int head = blockIdx.x / pt, i0 = (blockIdx.x % pt) * 16;
  const int row0 = blockIdx.y * 16 * TJ;
  const int lc = blockIdx.z, l = l0 + lc;
  const int M = a.batch * a.T;
  const int wi = min(i0 + lr, half - 1);  // channels past the half are not stored
  const T* wx = w + (int64_t)l * w_stride + ((int64_t)head * dh + wi) * d;
  const T* wy = wx + (int64_t)half * d;
  const T* xr[TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j) xr[j] = x + (int64_t)min(row0 + j * 16 + lr, M - 1) * d;
  floatx4 ax[TJ], ay[TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j) ax[j] = ay[j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
  for (int k0 = wave * 16; k0 < d; k0 += 16 * kGenWaves) {
    const int k = k0 + 4 * lg, n = d - k;  // VEC: n >= 4 or n <= 0
    floatx4 vx = {0.f, 0.f, 0.f, 0.f}, vy = vx, vb[TJ];
#pragma unroll
    for (int j = 0; j < TJ; ++j) vb[j] = vx;
    if (n > 0) {
      vx = ld4<VEC>(wx + k, n);
      vy = ld4<VEC>(wy + k, n);
#pragma unroll
      for (int j = 0; j < TJ; ++j) vb[j] = ld4<VEC>(xr[j] + k, n);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        ax[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vx[e], vb[j][e], ax[j], 0, 0, 0);
        ay[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vy[e], vb[j][e], ay[j], 0, 0, 0);
      }
  }
#pragma unroll
  for (int j = 0; j < TJ; ++j) {
    red[wave][0][j][lane] = ax[j];
    red[wave][1][j][lane] = ay[j];
  }
  __syncthreads();
  // lane l of a tile: channels i0 + 4 (l / 16) .. + 3 of token l % 16
  const int kind = head < g.Hq ? 0 : (head < g.Hq + g.Hkv ? 1 : 2);  // Q, K, V
  for (int e = tid; e < TJ * 64; e += 64 * kGenWaves) {
    const int j = e >> 6, el = e & 63;
    const int row = row0 + j * 16 + (el & 15), i = i0 + 4 * (el >> 4);
    if (row >= M || i >= half) continue;
    floatx4 xv = red[0][0][j][el], yv = red[0][1][j][el];
#pragma unroll
    for (int q = 1; q < kGenWaves; ++q) {
      xv += red[q][0][j][el];
      yv += red[q][1][j][el];
    }
    const int sq = row / a.T, t = row % a.T;
    const SeqDesc sd = a.seq[sq];
    const int u = sd.n_before + t;
    float xo[4] = {xv[0], xv[1], xv[2], xv[3]}, yo[4] = {yv[0], yv[1], yv[2], yv[3]};
    if (kind < 2) {
      const float* cr = g.rope_cos + (int64_t)(sd.pos0 + u) * half + i;
      const float* sr = g.rope_sin + (int64_t)(sd.pos0 + u) * half + i;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        xo[q] = xv[q] * cr[q] - yv[q] * sr[q];
        yo[q] = xv[q] * sr[q] + yv[q] * cr[q];
      }
    }
    T* p;
    if (kind == 0) {
      p = qbuf + ((int64_t)lc * M + row) * (g.Hq * dh) + head * dh + i;
    } else {
      const int hk = kind == 1 ? head - g.Hq : head - g.Hq - g.Hkv;
      const int32_t blk = g.tables[(int64_t)sd.slot * g.max_blocks + u / g.B];
      p = (T*)g.pool + (int64_t)blk * g.block_elems + tile_off(g, l, kind - 1, hk, u % g.B) + i;
    }
    st4(p, xo);
    st4(p + half, yo);
  }
}

// grid (batch x vector tiles, Hkv, lc), block 64 NW (NW = blockDim / 64);
// dynamic LDS: NW x 16 x (dh + 4 + 2) floats.  NC: 16-channel groups, at most
// (dh <= 16 NC).  S^T = K Q^T and O^T = V^T P^T as in the bf16 kernels: query
// vector in the matrix column, so that a lane's four scores (keys 4 (l / 16)
// + r of the tile) are the operands of the second product as they are.
template <typename T, int NC>
__global__ void __launch_bounds__(NC > 4 ? 512 : 1024)
k_attn_generic(PoolGeom g, const T* __restrict__ qbuf, AppendDesc a, T* __restrict__ o, int l0,
               float scale) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, NW = blockDim.x >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int G = g.Hq / g.Hkv, dh = g.dh, nc = dh / 16, M = a.batch * a.T;
  const int vecs = a.T * G, tiles = (vecs + 15) / 16;
  const int sq = blockIdx.x / tiles, vt = tiles - 1 - (int)(blockIdx.x % tiles);  // long first
  const int hk = blockIdx.y, lc = blockIdx.z, l = l0 + lc;
  const SeqDesc sd = a.seq[sq];
  const int v = min(vt * 16 + lr, vecs - 1);
  const int t = v / G, nkeys = sd.n_before + t + 1;
  const int n_all = sd.n_before + min(vt * 16 + 15, vecs - 1) / G + 1;  // keys of the tile's last
  const int n_first = sd.n_before + vt * 16 / G + 1;  // and of its first: seen by every vector
  const T* q = qbuf + (((int64_t)lc * M + sq * a.T + t) * g.Hq + hk * G + v % G) * dh;
  floatx4 qf[NC], oacc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    oacc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
    qf[c] = c < nc ? ld4<true>(q + c * 16 + 4 * lg, 4) : oacc[c];
  }
  const T* pool = (const T*)g.pool;
  const int32_t* trow = g.tables + (int64_t)sd.slot * g.max_blocks;
  const int64_t kbase = tile_off(g, l, 0, hk, 0), vbase = tile_off(g, l, 1, hk, 0);
  float m = -INFINITY, lsum = 0.f;
  // one tile of 16 keys; MASKED: some vector does not see all of them, and those
  // past the last read that one
  auto tile = [&](int k0, auto masked_c) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    const int key = MASKED ? min(k0 + lr, n_all - 1) : k0 + lr, kb = key / g.B, slot = key - kb * g.B;
    const int32_t blk = trow[kb];
    const T* kp = pool + (int64_t)blk * g.block_elems + kbase + (int64_t)slot * dh + 4 * lg;
    floatx4 kf[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (c < nc) kf[c] = ld4<true>(kp + c * 16, 4);
    // 0 * Inf and 0 * NaN are NaN: values that are not finite are kept from the
    // vectors that do not see their key (read as the keys are, beside them)
    bool odd = false;
    if constexpr (MASKED) {
      const T* ve = kp + (vbase - kbase);
#pragma unroll
      for (int c = 0; c < NC; ++c)
        if (c < nc) {
          const floatx4 f = ld4<true>(ve + c * 16, 4);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            odd |= (__float_as_uint(f[e]) & 0x7f800000u) == 0x7f800000u;
        }
      odd = __any(odd);
    }
    const T* vp[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int32_t vb = __shfl(blk, 4 * lg + r);
      const int vs = __shfl(slot, 4 * lg + r);
      vp[r] = pool + (int64_t)vb * g.block_elems + vbase + (int64_t)vs * dh + lr;
    }
    floatx4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (c < nc) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          sc = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][e], qf[c][e], sc, 0, 0, 0);
      }
    float p[4], mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = !MASKED || k0 + 4 * lg + r < nkeys ? sc[r] * scale : -INFINITY;
      mx = fmaxf(mx, p[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float mn = fmaxf(m, mx);
    const float mu = mn == -INFINITY ? 0.f : mn;  // no visible key yet
    float ps = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = __expf(p[r] - mu);
      ps += p[r];
    }
    ps += __shfl_xor(ps, 16);
    ps += __shfl_xor(ps, 32);
    const float alpha = __expf(m - mu);
    lsum = lsum * alpha + ps;
    m = mn;
#pragma unroll
    for (int c = 0; c < NC; ++c) oacc[c] *= alpha;
    if (MASKED && odd) {
      // a key at a time, into the columns that see it
#pragma unroll 1
      for (int i = 0; i < 16 && k0 + i < n_all; ++i) {
        const int r = i & 3;
        const bool own = lg == i >> 2, seen = k0 + i < nkeys;
        const T* vi = r == 0 ? vp[0] : r == 1 ? vp[1] : r == 2 ? vp[2] : vp[3];
        const float pi = own ? (r == 0 ? p[0] : r == 1 ? p[1] : r == 2 ? p[2] : p[3]) : 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c)
          if (c < nc) {
            const floatx4 t = __builtin_amdgcn_mfma_f32_16x16x4f32(
                own ? ld<T>(vi + c * 16) : 0.f, pi, oacc[c], 0, 0, 0);
            if (seen) oacc[c] = t;
          }
      }
      return;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (c < nc) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          oacc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(ld<T>(vp[r] + c * 16), p[r], oacc[c], 0,
                                                         0, 0);
      }
  };
  int k0 = wave * 16;
  for (; k0 + 16 <= n_first; k0 += 16 * NW) tile(k0, std::false_type{});
  for (; k0 < n_all; k0 += 16 * NW) tile(k0, std::true_type{});
  // combine the wavefronts: [NW][16][dh + 4] outputs, then m and l [NW][16]
  const int ldo = dh + 4;
  float* s_m = sm + NW * 16 * ldo;
  float* s_l = s_m + NW * 16;
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (c < nc) *(floatx4*)(sm + (wave * 16 + lr) * ldo + c * 16 + 4 * lg) = oacc[c];
  if (lg == 0) {
    s_m[wave * 16 + lr] = m;
    s_l[wave * 16 + lr] = lsum;
  }
  __syncthreads();
  const int c4n = dh / 4;
  for (int e = threadIdx.x; e < 16 * c4n; e += blockDim.x) {
    const int vv = e / c4n, c4 = e - vv * c4n, vi = vt * 16 + vv;
    if (vi >= vecs) continue;
    float mm = -INFINITY;
    for (int w = 0; w < NW; ++w) mm = fmaxf(mm, s_m[w * 16 + vv]);
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    float lt = 0.f;
    for (int w = 0; w < NW; ++w) {
      const float f = __expf(s_m[w * 16 + vv] - mm);
      lt += s_l[w * 16 + vv] * f;
      acc += *(const floatx4*)(sm + (w * 16 + vv) * ldo + c4 * 4) * f;
    }
    const float inv = 1.f / lt;
    const float out[4] = {acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
    st4(o + (((int64_t)l * M + sq * a.T + vi / G) * g.Hq + hk * G + vi % G) * dh + c4 * 4, out);
  }
}

template <typename T>
hipError_t run_qkv(const PoolGeom& g, const T* x, const T* w, int64_t w_stride,
                   const AppendDesc& a, T* qbuf, int l0, int lc, hipStream_t s) {
  const int M = a.batch * a.T;
  const int gx = (g.Hq + 2 * g.Hkv) * ((g.dh / 2 + 15) / 16);
  // rows and layers start on 4 elements
  const bool vec = g.d % 4 == 0 && w_stride % 4 == 0;
  // 16 rows a workgroup until that fills the device (256 CUs, four workgroups
  // each); from there on 64 rows, a quarter of the weight reads per row
  const bool wide = (int64_t)gx * ((M + 15) / 16) * lc > 1024;
  const int rows = wide ? 64 : 16;
  const dim3 grid(gx, (M + rows - 1) / rows, lc);
  auto kernel = wide ? (vec ? k_qkv_generic<T, 4, true> : k_qkv_generic<T, 4, false>)
                     : (vec ? k_qkv_generic<T, 1, true> : k_qkv_generic<T, 1, false>);
  kernel<<<grid, 64 * kGenWaves, 0, s>>>(g, x, w, w_stride, a, qbuf, l0);
  return hipGetLastError();
}

template <typename T>
hipError_t run_attn(const PoolGeom& g, const T* qbuf, const AppendDesc& a, T* o, int l0, int lc,
                    hipStream_t s) {
  const int vecs = a.T * (g.Hq / g.Hkv);
  const dim3 grid(a.batch * ((vecs + 15) / 16), g.Hkv, lc);
  const int64_t wgs = (int64_t)grid.x * grid.y * grid.z;
  // wavefronts: up to one per key tile; 16 where few workgroups read many
  // keys (and their registers allow it), 4 where the workgroups alone fill the
  // device
  int nw = wgs >= 2048 ? 4 : wgs < 256 && g.dh <= 64 ? 16 : 8;
  while (nw > 1 && nw * 16 >= 2 * a.max_keys) nw /= 2;
  const size_t lds = (size_t)nw * 16 * (g.dh + 6) * sizeof(float);
  const float scale = 1.0f / sqrtf((float)g.dh);
  auto kernel = g.dh <= 64 ? k_attn_generic<T, 4>
                : g.dh <= 128 ? k_attn_generic<T, 8>
                              : k_attn_generic<T, 16>;
  kernel<<<grid, 64 * nw, lds, s>>>(g, qbuf, a, o, l0, scale);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_qkv_generic(const PoolGeom& g, int dtype, const void* x, const void* w,
                              int64_t w_stride, const AppendDesc& a, void* qbuf, int l0, int lc,
                              hipStream_t s) {
  if (dtype == KV_DTYPE_BF16)
    return run_qkv(g, (const uint16_t*)x, (const uint16_t*)w, w_stride, a, (uint16_t*)qbuf, l0,
                   lc, s);
  return run_qkv(g, (const float*)x, (const float*)w, w_stride, a, (float*)qbuf, l0, lc, s);
}

hipError_t launch_attn_generic(const PoolGeom& g, int dtype, const void* qbuf,
                               const AppendDesc& a, void* o, int l0, int lc, hipStream_t s) {
  if (dtype == KV_DTYPE_BF16)
    return run_attn(g, (const uint16_t*)qbuf, a, (uint16_t*)o, l0, lc, s);
  return run_attn(g, (const float*)qbuf, a, (float*)o, l0, lc, s);
}

}  // namespace kvs
