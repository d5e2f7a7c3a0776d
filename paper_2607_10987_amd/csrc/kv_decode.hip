// Decode attention (a few new tokens per sequence) over the paged cache on
// MFMA, split over key chunks, reading each shared block once for the whole
// batch.
//
// Forked agents share the blocks of their common context (same physical ids
// in their block tables).  The keys of a call are cut into chunks of ck
// positions (decode_form below).  k_decode_plan (one workgroup per chunk)
// cuts a chunk into work units: the members whose blocks agree from the
// chunk's start share one unit up to the block where the first of them
// diverges, and what each has after that is a unit of its own (or of the
// members that agree to the end).  The grouping is the same for every layer
// and KV head, so it is computed once per call.
//
// A chunk used to be one unit only where all its blocks agreed, so a fork
// inside it made every member read the whole chunk: 32 agents on a ragged
// 6007-token context (8B shape, 32 layers) took 703 us per step against 251
// at 6144 tokens.
//
// The stream kernels run one wavefront per work item with no workgroup
// barriers: a wavefront streams the unit's K/V rows once, 32 keys at a time,
// through a ring of LDS stages filled by direct global->LDS copies, and scores
// all of the group's query vectors (members x T tokens x the G query heads of
// the KV head) with MFMA in the transposed layout of the prefill kernel (query
// vector in the MFMA column, softmax state lane-local, V^T operands by
// transposed LDS reads).  Per (query vector, unit) it writes a partial (running
// max m, running sum l, unnormalised output o); k_decode_merge combines the
// partials of a query with the usual log-sum-exp rescaling.  A unit's record
// carries its block ids, read with scalar loads one stage ahead of the copies.
//
// k_decode_pers is persistent: one workgroup per resident slot walks a
// static list of (unit, layer, KV head) items, largest first, and keeps its
// stage ring running across items, so the copy latency is paid once per
// workgroup rather than once per item (a stream-only probe that read every
// unit twice without a restart took 1.9x, not 2x, the time of one pass); a
// switch between items still costs about one refill of the ring.  It takes
// the units of more than 32 query vectors in calls of 65 to 256 (four or
// eight wavefronts sharing the ring).  k_decode_stream runs one wavefront per
// (unit, query slice of 64 vectors, KV head, layer) for the rest; the slices
// of a unit are launched on one XCD, so the later ones find the keys in its
// L2.
#include <algorithm>
#include <cmath>

#include "kv_dma.h"
#include "kv_fast.h"

namespace kvs {

bool attn_mfma_ok(const PoolGeom& g, int dtype, const AppendDesc& a);

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef short v4s __attribute__((ext_vector_type(4)));
#define KV_LDS4(p) ((__attribute__((address_space(3))) v4s*)(p))
// memory that no kernel of the same launch writes: uniform reads become
// scalar loads, which leave the copies' vmcnt order alone
typedef const __attribute__((address_space(4))) int32_t cint;

constexpr int kDh = 128;
constexpr int kCK = 1024;              // keys per chunk of the smallest layout
constexpr int kKT = 32;                // keys per pipeline stage
constexpr int kStage = 2 * kKT * kDh;  // elements per stage: K rows, then V rows
constexpr int kPart = kDh + 4;         // floats per partial: m, l, pad, pad, o[128]
constexpr int kUnitHdr = 4;            // words before a unit's block ids
// Shared keys x (members - 1) below which a diverging group is not cut at
// the divergence (the cut adds a unit and a partial per member).
constexpr int kMinShared = 64;

// A work unit is kUnitHdr + ck / B words: key0, nk, member mask (low, high),
// block ids.  The members in the mask read keys key0 .. key0 + nk - 1 of
// their states through these blocks (0 past the last).

// How a call's keys are cut.  Chunk c has one or two lists of units: list c,
// and with `split` list nch + c, which holds what follows a divergence
// inside the chunk.  A member is in at most one unit of a list, so a list is
// also the slot of the member's partial.  Units of at least big_members
// members come first in a list and are counted apart (n_units[list], then
// n_units[lists + list] for the others), since another kernel takes them.
struct DecodeForm {
  int ck, nch, lists, split;
  int unit_words, big_members;
};

// Reductions over lanes l and l ^ 32 (the two halves of a token's keys) with
// v_permlane32_swap, which leaves v[l % 32] and v[l % 32 + 32] in every lane.
__device__ inline float max_xor32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                  false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float sum_xor32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                  false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// LDS slot of chunk c of key row r: c ^ kswz(r) for K (read 16 rows at one
// chunk), c ^ vswz(r) for V (read transposed, 8 rows x 4 adjacent chunks);
// both spread each read over all bank groups.
__device__ inline int kswz(int r) { return r & 15; }
__device__ inline int vswz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }

__device__ inline uint32_t pack2(float a, float b) {
  const __bf16 x = (__bf16)a, y = (__bf16)b;
  return (uint32_t)__builtin_bit_cast(uint16_t, x) | ((uint32_t)__builtin_bit_cast(uint16_t, y) << 16);
}

// grid (nch), block 1024; dynamic LDS: batch * (ck / B) ints.
// Writes the units of chunk c to lists c and (split) nch + c of `units`, the
// lists' lengths (big units, others) to n_units, and to late[c] the members
// that have a unit in list nch + c.
//
// Latency-bound (a few hundred table words per workgroup).  The members are
// compared in parallel: a lane per member for the first blocks, a wavefront
// per member for its blocks.  One lane-per-group pass over the members with
// shuffles took 85 us at 32 members that all diverge, this one 11.
constexpr int kPlanThreads = 1024;

__global__ void __launch_bounds__(kPlanThreads)
k_decode_plan(PoolGeom g, AppendDesc a, int32_t* __restrict__ units, int* __restrict__ n_units,
              unsigned long long* __restrict__ late, DecodeForm f) {
  extern __shared__ int s_rows[];  // [batch][ck / B]: each member's block ids in the chunk, or -1
  __shared__ int s_nk[KV_MAX_BATCH], s_lead[KV_MAX_BATCH], s_pre[KV_MAX_BATCH];
  __shared__ int s_max[KV_MAX_BATCH], s_cnt[KV_MAX_BATCH], s_tail[KV_MAX_BATCH];
  __shared__ unsigned long long s_head_m[KV_MAX_BATCH], s_own_m[KV_MAX_BATCH];
  __shared__ int s_who[2][KV_MAX_BATCH];   // leader of list entry i
  __shared__ int s_len[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int NW = kPlanThreads / 64;
  const int c = blockIdx.x, b = a.batch, T = a.T;
  const int c0 = c * f.ck;
  const int nbc = f.ck >> g.b_shift;
  const int jb0 = c0 >> g.b_shift;
  // a wavefront per member, so that its descriptor is read once
#pragma unroll 4
  for (int m = wave; m < b; m += NW) {
    const int nb = (a.seq[m].n_before + T + g.B - 1) >> g.b_shift;
    const int32_t* trow = g.tables + (int64_t)a.seq[m].slot * g.max_blocks + jb0;
    for (int j = lane; j < nbc; j += 64) s_rows[m * nbc + j] = jb0 + j < nb ? trow[j] : -1;
  }
  if (tid < b) {
    s_nk[tid] = max(0, min(f.ck, a.seq[tid].n_before + T - c0));
    s_head_m[tid] = s_own_m[tid] = 0;
    s_pre[tid] = 0x7fffffff;
    s_max[tid] = 0;
    s_cnt[tid] = 0;
  }
  __syncthreads();
  // groups: the members with the same first block, led by the first of them
  if (tid < b) {
    int lead = -1;
    if (s_nk[tid] > 0) {
      const int first = s_rows[tid * nbc];
      lead = tid;
#pragma unroll 8
      for (int j = b - 1; j >= 0; --j)  // (a member without keys here has row -1)
        if (s_rows[j * nbc] == first) lead = j;
      atomicOr(&s_head_m[lead], 1ull << tid);
    }
    s_lead[tid] = lead;
  }
  __syncthreads();
  // keys a group's members have in common from the chunk's start
  for (int m = wave; m < b; m += NW) {
    const int lead = s_lead[m];
    if (lead < 0) continue;  // wavefront-uniform
    int q = nbc;
    for (int j0 = 0; j0 < nbc && q == nbc; j0 += 64) {
      const int j = j0 + lane;
      const uint64_t d = __ballot(j < nbc && s_rows[lead * nbc + j] != s_rows[m * nbc + j]);
      if (d) q = j0 + __builtin_ctzll(d);
    }
    if (lane == 0) {
      atomicMin(&s_pre[lead], min(q << g.b_shift, min(s_nk[m], s_nk[lead])));
      atomicMax(&s_max[lead], s_nk[m]);
      atomicAdd(&s_cnt[lead], 1);
    }
  }
  __syncthreads();
  // where each group is cut: nowhere when its members agree to the end, at
  // the last whole common block, or (0) before its first key
  if (tid < b && s_lead[tid] == tid && s_pre[tid] < s_max[tid]) {
    const int pre = s_pre[tid] & ~(g.B - 1);
    s_pre[tid] = f.split && pre * (s_cnt[tid] - 1) >= kMinShared ? pre : 0;
  }
  __syncthreads();
  // after the cut: the first member whose blocks agree to the chunk's end
  for (int m = wave; m < b; m += NW) {
    const int lead = s_lead[m];
    const int nk = s_nk[m], pre = lead < 0 ? 0 : s_pre[lead];
    int t = -1;
    if (lead >= 0 && pre < nk) {
      t = m;
      const int p0 = pre >> g.b_shift, nb = (nk + g.B - 1) >> g.b_shift;
      uint64_t cand = __ballot(lane < m && s_lead[lane] == lead && s_nk[lane] == nk &&
                               s_rows[lane * nbc + p0] == s_rows[m * nbc + p0]);
      while (cand) {
        const int j = __builtin_ctzll(cand);
        uint64_t d = 0;
        for (int i0 = p0; i0 < nb && d == 0; i0 += 64) {
          const int i = i0 + lane;
          d = __ballot(i < nb && s_rows[j * nbc + i] != s_rows[m * nbc + i]);
        }
        if (d == 0) {
          t = j;
          break;
        }
        cand &= cand - 1;
      }
    }
    if (lane == 0) {
      s_tail[m] = t;
      if (t >= 0) atomicOr(&s_own_m[t], 1ull << m);
    }
  }
  __syncthreads();
  if (wave == 0) {
    // (every lane takes part in the ballots below; only members have units)
    const bool in = lane < b;
    const int lead = in ? s_lead[lane] : -1, tail = in ? s_tail[lane] : -1;
    const int pre = lead >= 0 ? s_pre[lead] : 0;
    const bool head = lead == lane && pre > 0;  // leads a common unit
    const bool own = tail >= 0 && tail == lane;  // leads a unit after the cut
    const uint64_t m_head = in ? s_head_m[lane] : 0, m_own = in ? s_own_m[lane] : 0;
    const uint64_t below = lane ? ~0ull >> (64 - lane) : 0ull;
    int n_big[2];
    auto put = [&](int list, bool ok, int key0, int nk, uint64_t mask) {
      const bool big = __popcll(mask) >= f.big_members;
      const uint64_t mb = __ballot(ok && big), mo = __ballot(ok && !big);
      if (lane == 0) s_len[list] = __popcll(mb) + __popcll(mo);
      n_big[list] = __popcll(mb);
      if (!ok) return;
      const int idx = big ? __popcll(mb & below) : __popcll(mb) + __popcll(mo & below);
      int32_t* up = units + (int64_t)((list * f.nch + c) * b + idx) * f.unit_words;
      up[0] = key0;
      up[1] = nk;
      up[2] = (int32_t)(uint32_t)mask;
      up[3] = (int32_t)(uint32_t)(mask >> 32);
      s_who[list][idx] = lane;
    };
    put(0, head || (own && pre == 0), c0, head ? pre : (in ? s_nk[lane] : 0),
        head ? m_head : m_own);
    put(1, own && pre > 0, c0 + pre, in ? s_nk[lane] - pre : 0, m_own);
    const uint64_t lt = __ballot(tail >= 0 && pre > 0);
    if (lane == 0) {
      n_units[c] = n_big[0];
      n_units[f.lists + c] = s_len[0] - n_big[0];
      if (f.split) {
        n_units[f.nch + c] = n_big[1];
        n_units[f.lists + f.nch + c] = s_len[1] - n_big[1];
        late[c] = lt;
      }
    }
  }
  __syncthreads();
  for (int list = 0; list < 2; ++list)
    for (int q = wave; q < s_len[list]; q += NW) {
      const int m = s_who[list][q];
      const int pre = s_pre[s_lead[m]];
      const int p0 = list ? pre >> g.b_shift : 0;
      int32_t* up = units + (int64_t)((list * f.nch + c) * b + q) * f.unit_words + kUnitHdr;
      for (int j = lane; j < nbc; j += 64)
        up[j] = p0 + j < nbc ? max(s_rows[m * nbc + p0 + j], 0) : 0;
    }
}

// Which chunk holds unit u of the concatenated per-chunk unit lists, and the
// unit's index within it.  Wave-uniform.
__device__ inline void locate_unit(const int* __restrict__ n_units, int n_chunks, int u,
                                   int* chunk, int* idx) {
  const int lane = threadIdx.x & 63;
  int run = 0;
  *chunk = -1;
  for (int cb = 0; cb < n_chunks; cb += 64) {
    const int v = cb + lane < n_chunks ? n_units[cb + lane] : 0;
    int inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int t = __shfl_up(inc, d);
      if (lane >= d) inc += t;
    }
    const uint64_t hit = __ballot(v > 0 && run + inc - v <= u && u < run + inc);
    if (hit) {
      const int q = __builtin_ctzll(hit);
      *chunk = cb + q;
      *idx = u - run - __shfl(inc - v, q);
      return;
    }
    run += __shfl(inc, 63);
  }
}

// Wait until this wavefront's copies of the stage about to be read have
// landed: a wavefront's copies complete in issue order and it issues
// 2 * (kKT / 4) / NW copies of each stage (NW wavefronts share the copies),
// so at most `ahead` newer stages may still be pending (ahead <= 4).  Memory
// operations issued after the stage only lengthen the wait.
template <int NW = 1>
__device__ inline void wait_stage(int ahead) {
  constexpr int per = 2 * (kKT / 4) / NW;
  if (ahead >= 4)
    wait_vmcnt<(4 * per < 63 ? 4 * per : 63)>();
  else if (ahead == 3)
    wait_vmcnt<3 * per>();
  else if (ahead == 2)
    wait_vmcnt<2 * per>();
  else if (ahead == 1)
    wait_vmcnt<per>();
  else
    wait_vmcnt<0>();
}

// Block ids of a stage: 32 keys lie in one block, or two of 16 keys.
struct StageIds {
  int lo, hi;
};
__device__ inline StageIds stage_ids(const PoolGeom& g, cint* blk, int tile) {
  const int k0 = tile * kKT;
  return {blk[k0 >> g.b_shift], blk[(k0 + kKT / 2) >> g.b_shift]};
}

// Copies of one stage (keys [32 tile, 32 tile + 32) of a unit): 8 copies of
// 1 KiB (4 key rows, all in one block since B >= 16) per operand, block base
// in scalar registers, non-temporal (each byte is read once per call).
// pool_kv = the pool plus the offset of this (layer, KV head)'s K tile in a
// block.  Rows past the unit's last key read slots of a real block; their
// scores are masked and their V rows zeroed in LDS before use.
// With NW > 1 wavefronts sharing the stage, wavefront w issues copies w, w +
// NW, ... of each operand.
template <int NW = 1>
__device__ inline void issue_stage(const PoolGeom& g, const char* pool_kv, int64_t kv_gap,
                                   StageIds ids, int tile, uint32_t stage_lds, int lane,
                                   int w = 0) {
#pragma unroll
  for (int jj = 0; jj < kKT / 4 / NW; ++jj) {
    const int j = w + jj * NW;
    const int key0 = tile * kKT + j * 4;
    const int id = j < kKT / 8 ? ids.lo : ids.hi;
    const char* kb = pool_kv + ((int64_t)id * g.block_elems + (key0 & (g.B - 1)) * kDh) * 2;
    const int r = j * 4 + (lane >> 4);
    const uint32_t ko = (lane >> 4) * (kDh * 2) + (((lane & 15) ^ kswz(r)) * 16);
    const uint32_t vo = (lane >> 4) * (kDh * 2) + (((lane & 15) ^ vswz(r)) * 16);
    lds_dma16_sv_nt(kb, ko, stage_lds + j * 1024);
    lds_dma16_sv_nt(kb + kv_gap, vo, stage_lds + kKT * kDh * 2 + j * 1024);
  }
}

// Q^T operands of query vectors q0 .. q0 + 32 RT - 1 of a unit whose members
// are the bits of `mask`: vector r = (member rank * T + token) * G + head.
// qrow = the token's row of the call (-1 past the unit's R vectors), qhead =
// its query head, qlim = the last of the unit's keys that it sees (negative:
// none).  For T = 1 that is the unit's last key, a member's newest at most.
template <int RT>
__device__ __attribute__((always_inline)) inline void load_q(
    const PoolGeom& g, const uint16_t* __restrict__ qbuf, const AppendDesc& a, uint64_t mask,
    int key0, int nk, int R, int q0, int gk, int lc, int lane, bf16x8 (&qf)[RT][8],
    int (&qrow)[RT], int (&qhead)[RT], int (&qlim)[RT]) {
  const int G = g.Hq / g.Hkv, hl = lane >> 5, col = lane & 31, T = a.T;
  const int M = a.batch * T;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int r = q0 + rt * 32 + col;
    const bool ok = r < R;
    const int tok = ok ? r / G : 0;
    const int mi = T == 1 ? tok : tok / T, t = tok - mi * T;
    uint64_t mm = mask;
    if ((mask & (mask + 1)) == 0)  // the first members of the batch: rank = member
      mm = 1ull << mi;
    else
      for (int i = 0; i < mi; ++i) mm &= mm - 1;
    const int m = ok ? __builtin_ctzll(mm) : 0;
    qrow[rt] = ok ? m * T + t : -1;
    qhead[rt] = gk * G + (ok ? r - tok * G : 0);
    qlim[rt] = T == 1 ? nk - 1 : min(nk - 1, a.seq[m].n_before + t - key0);
    const uint16_t* qp = qbuf + (((int64_t)lc * M + (ok ? qrow[rt] : 0)) * g.Hq + qhead[rt]) * kDh;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
      qf[rt][ks] = ok ? *(const bf16x8*)(qp + ks * 16 + hl * 8) : bf16x8{};
  }
}

template <int RT>
__device__ __attribute__((always_inline)) inline void clear_state(floatx16 (&oacc)[RT][4],
                                                                  float (&m_run)[RT],
                                                                  float (&l_run)[RT]) {
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    m_run[rt] = -INFINITY;
    l_run[rt] = 0.f;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
      for (int e = 0; e < 16; ++e) oacc[rt][mt][e] = 0.f;
  }
}

// One stage, keys [k0, k0 + 32) of a unit with nk keys, K rows then V rows
// at Ks: S^T = K Q^T, the online softmax in base 2 (the running max moves
// only when it grows by more than 8), O^T += V^T P^T with V^T operands by
// transposed LDS reads.  `two`: the second query tile holds vectors.  The
// first nk_all keys are seen by every vector.
template <int RT>
__device__ __attribute__((always_inline)) inline void attend_stage(
    uint16_t* Ks, int k0, int nk, int nk_all, bool two, const bf16x8 (&qf)[RT][8],
    const int (&qlim)[RT], floatx16 (&oacc)[RT][4], float (&m_run)[RT], float (&l_run)[RT],
    float qk_scale_log2, int lane) {
  const int hl = lane >> 5, col = lane & 31;
  uint16_t* Vs = Ks + kKT * kDh;
  const bool tail = k0 + kKT > nk_all;  // wave-uniform
  if (tail) {  // V rows of keys >= nk may hold anything: zero them
    for (int i = (nk - k0) * (kDh / 8) + lane; i < kKT * (kDh / 8); i += 64)
      *(uint4*)(Vs + i * 8) = make_uint4(0, 0, 0, 0);
  }

  floatx16 sacc[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int e = 0; e < 16; ++e) sacc[rt][e] = 0.f;
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    const bf16x8 kf = *(const bf16x8*)(Ks + col * kDh + (((ks * 2 + hl) ^ kswz(col)) * 8));
    sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[0][ks], sacc[0], 0, 0, 0);
    if (two)
      sacc[RT - 1] =
          __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[RT - 1][ks], sacc[RT - 1], 0, 0, 0);
  }
  bf16x8 pf[RT][2];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    if (rt > 0 && !two) break;
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      float sv = sacc[rt][e];
      if (tail) {
        const int kk = k0 + (e >> 2) * 8 + hl * 4 + (e & 3);
        if (kk > qlim[rt]) sv = -INFINITY;
      }
      sacc[rt][e] = sv;
      mx = fmaxf(mx, sv);
    }
    mx = max_xor32(mx) * qk_scale_log2;
    const float m_new = mx > m_run[rt] + 8.f ? mx : m_run[rt];
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    const bool moved =
        __builtin_amdgcn_readfirstlane((int)(__ballot(m_new != m_run[rt]) != 0)) != 0;
    float psum = 0.f;
#pragma unroll
    for (int hs = 0; hs < 2; ++hs) {
      float p[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        p[j] = __builtin_amdgcn_exp2f(fmaf(sacc[rt][hs * 8 + j], qk_scale_log2, -m_use));
        psum += p[j];
      }
      uint32_t wv[4] = {pack2(p[0], p[1]), pack2(p[2], p[3]), pack2(p[4], p[5]),
                        pack2(p[6], p[7])};
      pf[rt][hs] = __builtin_bit_cast(bf16x8, *(uint4*)wv);
    }
    if (moved) {
      const float alpha = __builtin_amdgcn_exp2f(m_run[rt] - m_use);
      l_run[rt] *= alpha;
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[rt][mt][e] *= alpha;
    }
    l_run[rt] += psum;
    m_run[rt] = m_new;
  }
  const int g4 = lane >> 4, li = lane & 15;
#pragma unroll
  for (int s4 = 0; s4 < 2; ++s4) {
    const int key_a = s4 * 16 + (g4 >> 1) * 4 + (li >> 2), key_b = key_a + 8;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const int dc = mt * 32 + (g4 & 1) * 16 + (li & 3) * 4;
      const int ch = dc >> 3, hf = dc & 7;
      const v4s r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          KV_LDS4(Vs + key_a * kDh + ((ch ^ vswz(key_a)) * 8) + hf));
      const v4s r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          KV_LDS4(Vs + key_b * kDh + ((ch ^ vswz(key_b)) * 8) + hf));
      const v4s vv[2] = {r0, r1};
      const bf16x8 vf = __builtin_bit_cast(bf16x8, vv);
      oacc[0][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[0][s4], oacc[0][mt], 0, 0, 0);
      if (two)
        oacc[RT - 1][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[RT - 1][s4],
                                                                   oacc[RT - 1][mt], 0, 0, 0);
    }
  }
}

// Partials (m, l, o) of a unit's query vectors for list c, layer lc.
template <int RT>
__device__ __attribute__((always_inline)) inline void write_partials(
    float* __restrict__ part, const PoolGeom& g, int M, int lc, int c, int n_chunks,
    const int (&qrow)[RT], const int (&qhead)[RT], const floatx16 (&oacc)[RT][4],
    const float (&m_run)[RT], const float (&l_run)[RT], int lane) {
  const int hl = lane >> 5;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const float lt = sum_xor32(l_run[rt]);
    if (qrow[rt] < 0) continue;
    float* pp = part + ((((int64_t)lc * M + qrow[rt]) * g.Hq + qhead[rt]) * n_chunks + c) * kPart;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *(float4*)(pp + 4 + mt * 32 + q * 8 + hl * 4) =
            make_float4(oacc[rt][mt][q * 4], oacc[rt][mt][q * 4 + 1], oacc[rt][mt][q * 4 + 2],
                        oacc[rt][mt][q * 4 + 3]);
    if (hl == 0) {
      pp[0] = m_run[rt];
      pp[1] = lt;
    }
  }
}

// Block 64, ns = query slices per unit.  ns = 0: grid (Hkv x lc, slots),
// workgroups (., y) take units y, y + slots, ...: every layer and head of a
// unit before the next unit, so that the long units (which come first) start
// first and spread over all XCDs (unit-fastest order put 4 long units of 24 on
// the same 4 of 8 XCDs: 475 against 173 us for 16 agents x 6007 keys, 8B
// shape).  ns >= 1: grid (slots x ns, Hkv x lc), unit-fastest, slots a
// multiple of 8 for ns > 1, and x = (s / 8) * 8 ns + q * 8 + s % 8 takes
// slice q of units s, s + slots, ..., so all slices of a unit have the same
// x mod 8 (XCD).
// RT = query-vector tiles of 32 per slice (at most 32 RT vectors); S = LDS
// stages (S - 1 in flight while one is consumed).
template <int RT, int S>
__global__ void __launch_bounds__(64)
k_decode_stream(PoolGeom g, const uint16_t* __restrict__ qbuf, AppendDesc a,
                const int32_t* __restrict__ units, const int* __restrict__ n_big,
                float* __restrict__ part, int n_chunks, int unit_words, int l0,
                float qk_scale_log2, int ns) {
  static_assert(S >= 2 && S <= 4, "stages");
  __shared__ __attribute__((aligned(16))) uint16_t smem[S * kStage];
  const int lane = threadIdx.x;
  const int hl_i = ns == 0 ? blockIdx.x : blockIdx.y;
  const int gk = hl_i % g.Hkv, lc = hl_i / g.Hkv, layer = l0 + lc;
  const int G = g.Hq / g.Hkv, b = a.batch, M = b * a.T;
  const int64_t koff = tile_off(g, layer, 0, gk, 0), voff = tile_off(g, layer, 1, gk, 0);
  const char* pool_kv = (const char*)g.pool + koff * 2;
  const uint32_t lds0 = lds_addr(smem);
  const int64_t kv_gap = (voff - koff) * 2;  // bytes from a K row to its V row

  const int* n_units = n_big + n_chunks;  // the lists' other units
  const int x = ns == 0 ? blockIdx.y : blockIdx.x;
  const int slot = ns <= 1 ? x : (x / (8 * ns)) * 8 + (x & 7);
  const int qs = ns <= 1 ? 0 : (x >> 3) % ns;
  const int stride = ns == 0 ? gridDim.y : gridDim.x / ns;
  // one pass over the unit counts: their total, and the chunk and index of
  // this wavefront's first unit
  int total = 0, c_first = -1, gi_first = 0;
  for (int cb = 0; cb < n_chunks; cb += 64) {
    const int v = cb + lane < n_chunks ? n_units[cb + lane] : 0;
    int inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int tv = __shfl_up(inc, d);
      if (lane >= d) inc += tv;
    }
    const uint64_t hit = __ballot(v > 0 && total + inc - v <= slot && slot < total + inc);
    if (c_first < 0 && hit) {
      const int q = __builtin_ctzll(hit);
      c_first = cb + q;
      gi_first = slot - total - __shfl(inc - v, q);
    }
    total += __shfl(inc, 63);
  }
  total = __builtin_amdgcn_readfirstlane(total);
  for (int u = slot; u < total; u += stride) {
    int c = c_first, gi = gi_first;
    if (u != slot) locate_unit(n_units, n_chunks, u, &c, &gi);
    c = __builtin_amdgcn_readfirstlane(c);
    gi = __builtin_amdgcn_readfirstlane(gi);
    gi += ((cint*)n_big)[c];
    cint* up = (cint*)(units + (int64_t)(c * b + gi) * unit_words);
    const int key0 = up[0], nk = up[1];
    const uint64_t mask = ((uint64_t)(uint32_t)up[3] << 32) | (uint32_t)up[2];
    cint* blk = up + kUnitHdr;
    const int R = __popcll(mask) * a.T * G;  // query vectors of the unit
    const int q0 = qs * 32 * RT;       // this slice's first query vector
    if (q0 >= R) continue;             // wave-uniform: a unit with fewer slices
    const bool two = RT > 1 && R - q0 > 32;

    // the first stages go out before the query vectors are read, so that the
    // two latencies overlap (the wait for the queries below also waits for
    // these copies, which the first stage needs anyway)
    const int n_tiles = (nk + kKT - 1) / kKT;
    for (int st = 0; st < S - 1 && st < n_tiles; ++st)
      issue_stage(g, pool_kv, kv_gap, stage_ids(g, blk, st), st, lds0 + st * kStage * 2, lane);
    StageIds ids = stage_ids(g, blk, min(S - 1, n_tiles - 1));  // of the next stage to issue
    bf16x8 qf[RT][8];
    int qrow[RT], qhead[RT], qlim[RT];
    load_q<RT>(g, qbuf, a, mask, key0, nk, R, q0, gk, lc, lane, qf, qrow, qhead, qlim);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) settle(qf[rt][ks]);

    floatx16 oacc[RT][4];
    float m_run[RT], l_run[RT];
    clear_state<RT>(oacc, m_run, l_run);
    for (int t = 0; t < n_tiles; ++t) {
      wait_stage(min(S - 2, n_tiles - 1 - t));
      // stage (t - 1) % S was consumed in the previous iteration
      if (t + S - 1 < n_tiles) {
        issue_stage(g, pool_kv, kv_gap, ids, t + S - 1, lds0 + ((t + S - 1) % S) * kStage * 2,
                    lane);
        ids = stage_ids(g, blk, min(t + S, n_tiles - 1));
      }
      attend_stage<RT>(smem + (t % S) * kStage, t * kKT, nk, nk - a.T + 1, two, qf, qlim, oacc,
                       m_run, l_run, qk_scale_log2, lane);
    }
    write_partials<RT>(part, g, M, lc, c, n_chunks, qrow, qhead, oacc, m_run, l_run, lane);
  }
}

// Unit counts of up to 64 * kNR lists in registers (count and inclusive
// prefix of chunk 64 r + lane), so that a wavefront finds the chunk and
// index of any unit without a memory access.
constexpr int kNR = 4;
constexpr int kPersMaxChunks = 64 * kNR;

struct UnitIndex {
  int v[kNR], inc[kNR];
};

__device__ inline int index_units(const int* __restrict__ n_units, int n_chunks, int lane,
                                  UnitIndex& ix) {
  int run = 0;
#pragma unroll
  for (int r = 0; r < kNR; ++r) {
    const int v = 64 * r + lane < n_chunks ? n_units[64 * r + lane] : 0;
    int inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int tv = __shfl_up(inc, d);
      if (lane >= d) inc += tv;
    }
    ix.v[r] = v;
    ix.inc[r] = run + inc;
    run += __shfl(inc, 63);
  }
  return __builtin_amdgcn_readfirstlane(run);
}

__device__ inline void find_unit(const UnitIndex& ix, int u, int* c, int* gi) {
  int cc = 0, gg = 0;
#pragma unroll
  for (int r = 0; r < kNR; ++r) {
    const uint64_t hit = __ballot(ix.v[r] > 0 && ix.inc[r] - ix.v[r] <= u && u < ix.inc[r]);
    if (hit) {
      const int q = __builtin_ctzll(hit);
      cc = 64 * r + q;
      gg = u - __shfl(ix.inc[r] - ix.v[r], q);
    }
  }
  *c = __builtin_amdgcn_readfirstlane(cc);
  *gi = __builtin_amdgcn_readfirstlane(gg);
}

// A work item: one unit x one layer x one KV head.
struct DecodeItem {
  int c, lc, gk, key0, nk, n_tiles;
  uint64_t mask;
  const char* pool_kv;
  cint* blk;
};

// grid (W), block 64 NW, units of at most 32 RT NW query vectors, at most
// kPersMaxChunks lists.  Persistent: workgroup w takes items w, w + W, w +
// 2W, ... of the list (unit, layer, KV head) in that order, units in list
// order, so that the full chunks of a shared context come first and the
// short units after a divergence fill the end.  The NW wavefronts of a
// workgroup share one LDS stage ring (each issues its share of every stage's
// copies; a barrier per stage makes the stage visible to all and frees the
// slot consumed before it) and each scores 32 RT of the unit's query vectors,
// so that a deep ring and the matrix cores of several SIMDs serve the same
// bytes.  The ring runs across items: the first stages of the next item are
// issued while the current item's last stages are consumed, so a workgroup
// pays the copy latency once, not once per item.  The next item's query
// vectors (loaded at the start of the current item) are waited for only at
// the switch between items, the one point where the compiler drains a
// wavefront's memory operations; unit records come through scalar loads.
template <int NW, int RT, int S>
__global__ void __launch_bounds__(64 * NW)
k_decode_pers(PoolGeom g, const uint16_t* __restrict__ qbuf, AppendDesc a,
              const int32_t* __restrict__ units, const int* __restrict__ n_units,
              float* __restrict__ part, int n_chunks, int unit_words, int l0, int lcn,
              float qk_scale_log2) {
  static_assert(S >= 2 && S <= 6, "stages");
  static_assert(NW == 4 || NW == 8, "wavefronts per workgroup");
  __shared__ __attribute__((aligned(16))) uint16_t smem[S * kStage];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q0 = 32 * RT * wv;  // this wavefront's first query vector of a unit
  const int G = g.Hq / g.Hkv, b = a.batch, M = b * a.T;
  const uint32_t lds0 = lds_addr(smem);
  const int64_t kv_gap = (tile_off(g, 0, 1, 0, 0) - tile_off(g, 0, 0, 0, 0)) * 2;
  const int W = gridDim.x;

  UnitIndex ix;
  const int total = index_units(n_units, n_chunks, lane, ix);
  const int per_u = lcn * g.Hkv;
  const int n_items = total * per_u;
  int i = blockIdx.x;
  if (i >= n_items) return;  // workgroup-uniform

  auto make_item = [&](int j, DecodeItem& it) {
    const int u = j / per_u, r = j - u * per_u;
    it.lc = r / g.Hkv;
    it.gk = r - it.lc * g.Hkv;
    int gi;
    find_unit(ix, u, &it.c, &gi);
    cint* up = (cint*)(units + (int64_t)(it.c * b + gi) * unit_words);
    it.key0 = up[0];
    it.nk = up[1];
    it.mask = ((uint64_t)(uint32_t)up[3] << 32) | (uint32_t)up[2];
    it.n_tiles = (it.nk + kKT - 1) / kKT;
    it.pool_kv = (const char*)g.pool + tile_off(g, l0 + it.lc, 0, it.gk, 0) * 2;
    it.blk = up + kUnitHdr;
  };
  auto vectors = [&](const DecodeItem& it) { return __popcll(it.mask) * a.T * G; };

  DecodeItem cur, nxt{};
  bool has_nxt = i + W < n_items;
  bf16x8 qf[RT][8], qn[RT][8];
  int qrow[RT], qhead[RT], qlim[RT], qrow_n[RT], qhead_n[RT], qlim_n[RT];
  make_item(i, cur);
  if (has_nxt) make_item(i + W, nxt);
  load_q<RT>(g, qbuf, a, cur.mask, cur.key0, cur.nk, vectors(cur), q0, cur.gk, cur.lc, lane, qf,
             qrow, qhead, qlim);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) settle(qf[rt][ks]);

  int base = 0;    // stream index of cur's first stage
  int issued = 0;  // stages issued so far
  // block ids of stream stage s, if it is one of cur's or nxt's
  auto ids_of = [&](int s) {
    const int t = s - base;
    if (t < cur.n_tiles) return stage_ids(g, cur.blk, t);
    if (has_nxt) return stage_ids(g, nxt.blk, min(t - cur.n_tiles, nxt.n_tiles - 1));
    return StageIds{0, 0};
  };
  StageIds ids = ids_of(0);  // of stage `issued`
  // issue this wavefront's share of the next stage of the stream (cur's
  // stages, then nxt's) if any
  auto issue_next = [&]() {
    const int s = issued;
    const uint32_t sl = lds0 + (s % S) * kStage * 2;
    if (s - base < cur.n_tiles) {
      issue_stage<NW>(g, cur.pool_kv, kv_gap, ids, s - base, sl, lane, wv);
      ++issued;
    } else if (has_nxt && s - base - cur.n_tiles < nxt.n_tiles) {
      issue_stage<NW>(g, nxt.pool_kv, kv_gap, ids, s - base - cur.n_tiles, sl, lane, wv);
      ++issued;
    } else {
      return;
    }
    ids = ids_of(issued);
  };

  floatx16 oacc[RT][4];
  float m_run[RT], l_run[RT];
  for (;;) {
    // prefetch for the switch after this item: nxt's query vectors
    // (unconditional, so that no copy of a pending value lands before the
    // switch: no next item loads nothing)
    const bool has_nn = has_nxt && i + 2 * W < n_items;
    load_q<RT>(g, qbuf, a, has_nxt ? nxt.mask : 1, nxt.key0, nxt.nk, has_nxt ? vectors(nxt) : 0,
               q0, nxt.gk, nxt.lc, lane, qn, qrow_n, qhead_n, qlim_n);
    // top up the ring to S - 1 stages ahead; every slot written here was
    // consumed before the last barrier
#pragma unroll
    for (int st = 0; st < S - 1; ++st)
      if (issued - base < S - 1) issue_next();

    const int R = vectors(cur);
    const bool active = q0 < R;              // wavefront-uniform
    const bool two = RT > 1 && R - q0 > 32;
    clear_state<RT>(oacc, m_run, l_run);
    for (int t = 0; t < cur.n_tiles; ++t) {
      const int s = base + t;
      wait_stage<NW>(issued - s - 1);
      // every wavefront's copies of stage s are visible and every LDS access
      // of stage s - 1 (reads, tail zeroing) is done, so its slot may be
      // refilled
      lds_barrier();
      if (issued < s + S) issue_next();
      if (active)
        attend_stage<RT>(smem + (s % S) * kStage, t * kKT, cur.nk, cur.nk - a.T + 1, two, qf,
                         qlim, oacc, m_run, l_run, qk_scale_log2, lane);
    }
    if (!has_nxt) {
      write_partials<RT>(part, g, M, cur.lc, cur.c, n_chunks, qrow, qhead, oacc, m_run, l_run,
                         lane);
      return;
    }
    // the switch: the one wait for the prefetched values
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) settle(qn[rt][ks]);
    write_partials<RT>(part, g, M, cur.lc, cur.c, n_chunks, qrow, qhead, oacc, m_run, l_run,
                       lane);
    base += cur.n_tiles;
    cur = nxt;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      qrow[rt] = qrow_n[rt];
      qhead[rt] = qhead_n[rt];
      qlim[rt] = qlim_n[rt];
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) qf[rt][ks] = qn[rt][ks];
    }
    has_nxt = has_nn;
    if (has_nn) make_item(i + 2 * W, nxt);
    i += W;
    // the stage after cur's may be one of the new nxt's
    ids = ids_of(issued);
  }
}

// grid (M * Hq, lc), block 64: combine the partials of one query.  The
// query's units are lists 0 .. nc - 1 and, with split lists, those of lists
// nch + c whose `late` mask holds its member; their list indices and weights
// exp2(m - max) go through LDS.  Lane i owns output channels 2i, 2i + 1.
__global__ void __launch_bounds__(64)
k_decode_merge(PoolGeom g, AppendDesc a, const float* __restrict__ part,
               const unsigned long long* __restrict__ late, DecodeForm f,
               uint16_t* __restrict__ o, int l0) {
  __shared__ float s_w[64];
  __shared__ int s_i[64];
  const int sh = blockIdx.x, lc = blockIdx.y, lane = threadIdx.x;
  const int row = sh / g.Hq, h = sh % g.Hq;
  const int M = a.batch * a.T;
  const int m = row / a.T;
  const int nc = (a.seq[m].n_before + a.T + f.ck - 1) / f.ck;
  const float* pp = part + (((int64_t)lc * M + row) * g.Hq + h) * f.lists * kPart;
  auto valid = [&](int i) {
    if (i < f.nch) return i < nc;
    return i < f.lists && ((late[i - f.nch] >> m) & 1);
  };
  float mx = -INFINITY;
  for (int i = lane; i < f.lists; i += 64)
    if (valid(i)) mx = fmaxf(mx, pp[(int64_t)i * kPart]);
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) mx = fmaxf(mx, __shfl_xor(mx, d));
  float lsum = 0.f;
  float2 acc = make_float2(0.f, 0.f);
  for (int i0 = 0; i0 < f.lists; i0 += 64) {
    const int i = i0 + lane;
    const bool ok = valid(i);
    const uint64_t vm = __ballot(ok);
    const int cn = __popcll(vm);
    if (ok) {
      const float w = exp2f(pp[(int64_t)i * kPart] - mx);
      lsum += pp[(int64_t)i * kPart + 1] * w;
      const int k = lane ? __popcll(vm & (~0ull >> (64 - lane))) : 0;
      s_w[k] = w;
      s_i[k] = i;
    }
    __syncthreads();
    const float* q = pp + 4 + 2 * lane;
    int k = 0;
    for (; k + 4 <= cn; k += 4) {
      const float2 v0 = *(const float2*)(q + (int64_t)s_i[k] * kPart);
      const float2 v1 = *(const float2*)(q + (int64_t)s_i[k + 1] * kPart);
      const float2 v2 = *(const float2*)(q + (int64_t)s_i[k + 2] * kPart);
      const float2 v3 = *(const float2*)(q + (int64_t)s_i[k + 3] * kPart);
      acc.x += v0.x * s_w[k] + v1.x * s_w[k + 1] + v2.x * s_w[k + 2] + v3.x * s_w[k + 3];
      acc.y += v0.y * s_w[k] + v1.y * s_w[k + 1] + v2.y * s_w[k + 2] + v3.y * s_w[k + 3];
    }
    for (; k < cn; ++k) {
      const float2 v = *(const float2*)(q + (int64_t)s_i[k] * kPart);
      acc.x += v.x * s_w[k];
      acc.y += v.y * s_w[k];
    }
    __syncthreads();
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) lsum += __shfl_xor(lsum, d);
  const float inv = 1.f / lsum;
  const int l = l0 + lc;
  *(uint32_t*)(o + (((int64_t)l * M + row) * g.Hq + h) * kDh + 2 * lane) =
      pack2(acc.x * inv, acc.y * inv);
}

}  // namespace

namespace {

constexpr int kMaxVec = 256;    // query vectors that one workgroup takes (8 wavefronts of 32)
// Query vectors up to which T > 1 calls run here: at more, the prefill
// attention's matrix-core rate counts for more than its idle rows (a batch of
// one over 5003 keys, 8B shape: 32 tokens 165 against 200 us, 64 tokens 363
// against 180).
constexpr int kMaxVecAppend = 128;

// `wide` = the form with split lists and chunks cut to fit the device; else
// the smallest layout (T = 1 only).
//
// Chunk size of the wide form.  A partial is 528 bytes written and read per
// (query vector, unit) against 512 bytes of keys and values per key, so
// chunks grow with the query vectors (16 keys per vector: partials an eighth
// of the traffic).  Within a factor of about 1.5 of that size the number of
// chunks is the one whose (chunk, layer, KV head) items best fill whole rounds
// of the workgroups that are resident for this many vectors, 5 (one
// wavefront), 4 (one, two query tiles), 2 (four) or 1 (eight) per CU, with a
// chunk costing its keys, its partials and about 32 keys to start.  (Rounds of
// the whole call: in a work area that cuts it into layer groups they are
// smaller.)  A batch of one has no shared blocks and its chunks are its only
// parallelism: about 512 (+5-10% against 1024).  The device's 256 CUs are a
// constant here: kv_scratch_bytes, which asks no device, has to arrive at the
// same form as the launch.
int64_t wide_keys(int64_t batch, int64_t vec) {
  return std::max<int64_t>(batch == 1 ? kCK / 2 : kCK, std::min<int64_t>(16 * vec, 4 * kCK));
}
int64_t wide_chunks(int64_t keys, int64_t ck) {
  return std::max<int64_t>(1, (keys + ck / 2) / ck);
}
// k_decode_plan holds a chunk's block ids of every member in LDS, beside 3080
// bytes of its own in the 160 KiB of a CU: the bound on a chunk of many members
// (64 of them, blocks of 16: 9984 keys).  The largest chunk that the fit asks
// for is 2.5 times wide_keys, 10240 keys.
constexpr size_t kPlanLds = 156 * 1024;
size_t plan_lds(const PoolGeom& g, const AppendDesc& a, int64_t ck) {
  return (size_t)a.batch * (ck / g.B) * sizeof(int);
}
DecodeForm decode_form(const PoolGeom& g, const AppendDesc& a, bool wide) {
  DecodeForm f;
  f.ck = a.batch == 1 ? kCK / 2 : kCK;
  const int64_t G = g.Hq / g.Hkv, vec = (int64_t)a.batch * a.T * G;
  if (wide) {
    // One token of one state: all units are alike.  While 1024-key chunks need
    // at most two rounds of four workgroups per CU, the fit is to those (a fifth
    // resident one only takes bandwidth from the others) and may go down to 256
    // keys (few layers) or up to 1024: over five shapes of 16 to 640 (layer, KV
    // head) pairs and 20 key counts to 34816, 1.6% above the best of ten fixed
    // sizes on average, against 7% for 384 keys, 10% for 512.  Beyond two rounds
    // units drift apart and full rounds do not count: 384 keys up to four of them
    // (8B shape, 9000 keys, 4 steps: 811 us against 947 for three full rounds of
    // 768), then the fit below, near 512 (70B shape, 8000 keys, a step: 438
    // against 449 for 384).  Where the pool lies in memory moves these times by
    // up to 4%.
    const int64_t U = (int64_t)g.L * g.Hkv;
    const double kilo = (double)a.max_keys * U / (kCK * 1024.0);  // rounds of 1024-key units
    const bool one = a.batch == 1 && a.T == 1, few = one && kilo <= 2;
    const int64_t per_cu = few ? 4 : vec <= 32 ? 5 : vec <= 64 ? 4 : vec <= 128 ? 2 : 1;
    const int64_t slots = 256 * per_cu;
    const int64_t want = wide_keys(a.batch, vec);
    const int64_t unit = std::max(64, g.B);
    const int64_t n0 = wide_chunks(a.max_keys, want);
    double best = 0;
    int64_t ck = want;
    const int64_t n_lo = std::max<int64_t>(1, few ? n0 / 2 : 2 * n0 / 3);
    for (int64_t n = few ? 2 * n0 : n0 + (n0 + 1) / 2; n >= n_lo; --n) {
      const int64_t c = std::max<int64_t>(((a.max_keys + n - 1) / n + unit - 1) / unit * unit, 256);
      if (plan_lds(g, a, c) > kPlanLds) break;  // fewer chunks are larger still
      const int64_t nch = (a.max_keys + c - 1) / c;
      const int64_t rounds = (nch * U + slots - 1) / slots;
      const double fill = (double)(a.max_keys * U) / (double)(rounds * slots * c);
      const double rate = fill / (1.0 + (2.0 * vec + 32.0) / c);
      if (rate > best) {
        best = rate;
        ck = c;
      }
      n = nch;  // down to here the chunk is the same
    }
    f.ck = one && !few && kilo < 4 ? 384 : (int)ck;
  }
  f.nch = (a.max_keys + f.ck - 1) / f.ck;
  f.split = wide && a.batch > 1 ? 1 : 0;
  f.lists = f.split ? 2 * f.nch : f.nch;
  f.unit_words = kUnitHdr + (f.ck >> (g.b_shift < 0 ? 0 : g.b_shift));
  f.big_members = vec > 64 && vec <= kMaxVec && f.lists <= kPersMaxChunks
                      ? (int)(32 / (a.T * G) + 1)
                      : KV_MAX_BATCH + 1;
  return f;
}

size_t up256(size_t n) { return (n + 255) & ~size_t(255); }

size_t unit_bytes(const AppendDesc& a, const DecodeForm& f) {
  return up256((size_t)f.lists * a.batch * f.unit_words * sizeof(int32_t));
}
size_t count_bytes(const DecodeForm& f) { return up256((size_t)f.lists * 2 * sizeof(int)); }

}  // namespace

// T = 1: any batch (query slices of 64 vectors cover batch x G).
bool decode_mfma_ok(const PoolGeom& g, int dtype, const AppendDesc& a) {
  // ck % B == 0 with B >= 16 a power of two
  if (!(dtype == KV_DTYPE_BF16 && g.dh == kDh && a.batch <= KV_MAX_BATCH && g.B >= 16 &&
        g.b_shift >= 0 && (a.batch == 1 ? kCK / 2 : kCK) % g.B == 0))
    return false;
  if (a.T == 1) return true;
  // Appends: in the place of the prefill attention only, which rounds its
  // probabilities to bf16 as well.  What that does not cover (other head groups,
  // longer block tables) keeps the portable kernel's float32 ones.
  if (!attn_mfma_ok(g, dtype, a)) return false;
  const int G = g.Hq / g.Hkv;
  const DecodeForm f = decode_form(g, a, true);
  if ((int64_t)a.batch * a.T * G > kMaxVecAppend || f.lists > kPersMaxChunks) return false;
  // The prefill attention runs a round of 256 workgroups per 256
  // (sequence, KV head, layer), each 11 us and 1 us per 32 keys; this path
  // costs three launches, about 40 us, and the keys at about 5.5 TB/s.  8B
  // shape: a prefill of 16 tokens 12 against 31 us, 8 tokens over 5003 keys 207
  // against 139, 6 x 2 tokens over 5003 keys 1103 against 139.
  const double items = (double)a.batch * g.Hkv * g.L;
  const double rounds = ceil(items / 256);
  const double split = 40 + (double)a.max_keys * g.Hkv * g.L * 512 / 5.5e6;
  return split < rounds * (11 + a.max_keys / 32.0);
}

// Scratch of a call: the split-key partials of one layer, [M][Hq][lists][kPart]
// floats, and the work plan (units, list lengths, late masks).
void decode_scratch(const PoolGeom& g, const AppendDesc& a, bool wide, size_t* per_layer,
                    size_t* fixed) {
  const DecodeForm f = decode_form(g, a, wide);
  *per_layer = up256((size_t)a.batch * a.T * g.Hq * f.lists * kPart * sizeof(float));
  *fixed = unit_bytes(a, f) + count_bytes(f) +
           (f.split ? up256((size_t)f.nch * sizeof(uint64_t)) : 0);
}

void decode_query(const PoolGeom& g, const AppendDesc& a, bool wide, int64_t* out) {
  const DecodeForm f = decode_form(g, a, wide);
  out[0] = f.ck;
  out[1] = f.nch;
  out[2] = f.lists;
  out[3] = (int64_t)plan_lds(g, a, f.ck);
}

// The most that any call of up to `batch` states, `tokens` new tokens in all and
// max_keys keys takes.  The smallest layout has a formula; the wide form is
// asked for each number of rows, of one state and of several (how many only
// matters for the plan's LDS, far above the chunks of appends).  Its choice
// only changes where a multiple of 64 keys or a half step of wide_chunks is
// passed, so both ends of every 64 keys cover all key counts, from the most
// down to where a formula with the most chunks that it considers is no more
// than what was found.  That formula alone would ask for twice as much (8B
// shape, 16 agents, 33792 keys: 866 MB against 416; the smallest layout takes
// 285).
size_t decode_scratch_bound(const PoolGeom& g, int dtype, int64_t tokens, int64_t batch,
                            int64_t max_keys) {
  const int64_t L = g.L, Hq = g.Hq, G = g.Hq / g.Hkv;
  auto total = [&](int64_t rows, int64_t b, int64_t lists, int64_t ck) {
    return (size_t)L * (rows * Hq * lists * kPart * sizeof(float) + 256) +
           (size_t)lists * b * (kUnitHdr + ck / 16) * sizeof(int32_t) +
           (size_t)lists * (2 * sizeof(int) + sizeof(uint64_t)) + 4 * 256;
  };
  auto chunks = [&](int64_t ck) { return (max_keys + ck - 1) / ck; };
  size_t worst = std::max(total(1, 1, chunks(kCK / 2), kCK / 2),
                          total(batch, batch, chunks(kCK), kCK));
  AppendDesc a = {};
  auto wide = [&](int64_t b, int64_t T) {
    a.batch = (int32_t)b;
    a.T = (int32_t)T;
    const int64_t want = wide_keys(b, b * T * G);
    for (int64_t hi = (max_keys + 63) / 64 * 64; hi > 0; hi -= 64) {
      const int64_t n0 = wide_chunks(hi, want), n = b * T == 1 ? 2 * n0 : n0 + (n0 + 1) / 2;
      if (total(b * T, b, b > 1 ? 2 * n : n, 3 * want) <= worst) return;
      for (const int64_t keys : {std::max(T, hi - 63), std::min(max_keys, hi)}) {
        if (keys < T || keys > max_keys) continue;
        a.max_keys = (int32_t)keys;
        if (T > 1 && !attn_mfma_ok(g, dtype, a)) continue;  // too long a block table
        size_t per = 0, fixed = 0;
        decode_scratch(g, a, true, &per, &fixed);
        worst = std::max(worst, L * per + fixed);
      }
    }
  };
  a.batch = a.T = a.max_keys = 1;
  if (!decode_mfma_ok(g, dtype, a)) return worst;
  const bool appends = attn_mfma_ok(g, dtype, a);
  const int64_t most = std::min<int64_t>(batch, KV_MAX_BATCH);
  for (int64_t b = most; b >= 1; --b) wide(b, 1);
  const int64_t rows = appends ? std::min(tokens, (int64_t)kMaxVecAppend / G) : 0;
  for (int64_t r = rows; r > 1; --r) {
    wide(1, r);
    for (int64_t b = 2; r > most && b <= most; ++b)  // r <= most: as r states of a token
      if (r % b == 0) {
        wide(b, r / b);
        break;
      }
  }
  return worst;
}

namespace {
// Resident workgroups of k_decode_pers<NW, RT, S> on the current device: CUs
// x workgroups per CU (bounded by LDS and registers), cached per device.
template <int NW, int RT, int S>
int pers_slots() {
  static int cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (cache[dev] == 0) {
    int cus = 0, per = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per, reinterpret_cast<const void*>(&k_decode_pers<NW, RT, S>), 64 * NW, 0) !=
            hipSuccess)
      return 256;
    cache[dev] = std::max(1, cus * per);
  }
  return cache[dev];
}

template <int NW, int RT, int S>
void launch_pers(const PoolGeom& g, const void* qbuf, const AppendDesc& a, const int32_t* units,
                 const int* n_units, float* part, const DecodeForm& f, int l0, int lc, float sc,
                 int64_t items_max, hipStream_t s) {
  const int w = (int)std::min<int64_t>(pers_slots<NW, RT, S>(), items_max);
  k_decode_pers<NW, RT, S><<<w, 64 * NW, 0, s>>>(g, (const uint16_t*)qbuf, a, units, n_units, part,
                                                 f.lists, f.unit_words, l0, lc, sc);
}
}  // namespace

hipError_t launch_decode_attn(const PoolGeom& g, const void* qbuf, const AppendDesc& a, bool wide,
                              void* part_area, void* plan, int lc, int l0, hipStream_t s) {
  const int G = g.Hq / g.Hkv;
  const DecodeForm f = decode_form(g, a, wide);
  float* part = (float*)part_area;
  int32_t* units = (int32_t*)plan;
  int* n_units = (int*)((char*)plan + unit_bytes(a, f));
  unsigned long long* late = (unsigned long long*)((char*)n_units + count_bytes(f));
  if (l0 == 0) {  // the grouping holds for every layer group of the call
    k_decode_plan<<<f.nch, kPlanThreads, plan_lds(g, a, f.ck), s>>>(g, a, units, n_units, late, f);
  }
  const float sc = 1.4426950408889634f / sqrtf((float)kDh);
  int slots = std::min(f.nch * a.batch, 2 * f.nch + a.batch);
  const int vec = a.batch * a.T * G;
  const int64_t items_max = (int64_t)f.nch * a.batch * lc * g.Hkv;
  // Calls of 65 to 256 query vectors: their units of more than 32 by the
  // persistent form, four or eight wavefronts of 32 vectors per workgroup
  // sharing one stage ring (as units of one wavefront, 496 against 341 us for
  // 32 agents x 8192 keys, 8B shape; fewer vectors leave its wavefronts idle).
  if (f.big_members <= a.batch) {
    if (vec > 128)
      launch_pers<8, 1, 6>(g, qbuf, a, units, n_units, part, f, l0, lc, sc, items_max, s);
    else
      launch_pers<4, 1, 4>(g, qbuf, a, units, n_units, part, f, l0, lc, sc, items_max, s);
  }
  // The others: one wavefront per (unit, query slice of 64 vectors, KV head,
  // layer), two stages: with two query tiles 15% faster than three, with one
  // (five wavefronts a CU instead of three) 3-5% on short units and as fast on
  // long ones.  (A persistent form with one wavefront per slot was never
  // faster once long units start first: 170 against 144 us for 4 agents x
  // 1000 keys, 4 steps, 2860 against 2710 at 32768 keys, 8B shape.)
  const int few = f.big_members <= a.batch ? (f.big_members - 1) * a.T * G : vec;
  if (few == 0) return hipGetLastError();  // every unit is a big one
  // query slices of 64 vectors; a batch of one, whose units are all alike,
  // runs unit-fastest (5.58 against 5.98 ms for 8 steps over 34816 keys)
  int ns = (few + 63) / 64;
  if (ns == 1 && a.batch > 1) ns = 0;
  if (ns > 1) slots = (slots + 7) / 8 * 8;
  const dim3 grid = ns == 0 ? dim3(g.Hkv * lc, slots) : dim3(slots * ns, g.Hkv * lc);
  if (few <= 32)
    k_decode_stream<1, 2><<<grid, 64, 0, s>>>(g, (const uint16_t*)qbuf, a, units, n_units, part,
                                              f.lists, f.unit_words, l0, sc, ns);
  else
    k_decode_stream<2, 2><<<grid, 64, 0, s>>>(g, (const uint16_t*)qbuf, a, units, n_units, part,
                                              f.lists, f.unit_words, l0, sc, ns);
  return hipGetLastError();
}

hipError_t launch_decode_merge(const PoolGeom& g, const AppendDesc& a, bool wide, void* o,
                               const void* part, const void* plan, int l0, int lc,
                               hipStream_t s) {
  const DecodeForm f = decode_form(g, a, wide);
  const unsigned long long* late =
      (const unsigned long long*)((const char*)plan + unit_bytes(a, f) + count_bytes(f));
  dim3 grid(a.batch * a.T * g.Hq, lc);
  k_decode_merge<<<grid, 64, 0, s>>>(g, a, (const float*)part, late, f, (uint16_t*)o, l0);
  return hipGetLastError();
}

}  // namespace kvs
