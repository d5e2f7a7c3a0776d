// Block allocator kernels: the free ring, refcounts and block tables live in
// device memory and are only changed here.
//
// Semantics (the paper's metadata catalog: a block's refcount is the number of
// logical states that share it; KV-Fork aliases blocks by raising refcounts;
// KV-Evict frees a state's blocks, shared blocks surviving while referenced):
//  - allocation pops ids from the ring head in order (FIFO), so a sequence of
//    operations has exactly one resulting set of tables;
//  - release decrements a state's blocks in logical order and appends the ids
//    reaching zero to the ring tail in that order (a workgroup prefix scan
//    assigns ring slots, no atomics), states in the given order.
// Each kernel is a single workgroup or touches disjoint ids, so results are
// deterministic.  A mismatch with the host's expected counters sets the sticky
// status KV_ERR_INTERNAL and the kernel does nothing.  k_alloc also checks the
// host's copy-on-write decisions against the refcounts in both directions (a
// tail it copies must be shared, a partial tail it appends to in place must
// not be) and sets the same status when they disagree.
#include "kv_internal.h"

namespace kvs {

namespace {

constexpr int kMetaThreads = 256;
constexpr int kAllocThreads = 1024;
// k_release: 1024 threads where a state has more than three rounds of 256
// blocks (16 states of 2112: 118 -> 81 us), else 256, whose scan is cheaper
// (40 states of 20 blocks: 36 us against 60).
constexpr int kReleaseThreads = 1024;

__device__ inline bool fail_if(DevHeader* hdr, bool bad) {
  if (bad && threadIdx.x == 0) hdr->status = KV_ERR_INTERNAL;
  return bad;
}

// The requests' ring positions come from a prefix sum over them; copy-on-write
// runs a lane per request (several may leave the same tail: the decrements are
// atomic and each sees another count), then a wavefront per request draws its
// blocks.  One request after the other took 0.6 us each (64 requests: 44 us).
__global__ void __launch_bounds__(kAllocThreads)
k_alloc(DevHeader* hdr, int32_t* ring, int32_t* rc, int32_t* tables, int32_t max_blocks,
        int32_t P, int64_t head, AllocArgs a, int2* cow_pairs) {
  static_assert(KV_MAX_BATCH <= 64, "a lane per request");
  __shared__ int ok;
  __shared__ int64_t s_pos[KV_MAX_BATCH];  // first ring position after the request's copy-on-write
  __shared__ int32_t s_left[KV_MAX_BATCH];  // tail that the request's copy-on-write left, or -1
  __shared__ int any_cow;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool req = tid < a.n_req;
  if (wave == 0) {
    const int cow = req && a.req[lane].cow > 0;
    int64_t sum = req ? (int64_t)a.req[lane].count + cow : 0;
    const int64_t own = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int64_t t = __shfl_up((long long)sum, d);
      if (lane >= d) sum += t;
    }
    const int64_t need = __shfl((long long)sum, 63);
    if (req) {
      s_pos[lane] = head + sum - own + cow;
      s_left[lane] = -1;
    }
    const bool some = __ballot(cow) != 0;
    if (lane == 0) {
      any_cow = some;
      ok = hdr->status == 0 && hdr->head == head && hdr->tail - head >= need;
      if (ok) hdr->head = head + need;
    }
  }
  __syncthreads();
  if (fail_if(hdr, !ok)) return;
  if (req && a.req[tid].cow > 0) {
    const AllocReq q = a.req[tid];
    int32_t* tail = tables + (int64_t)q.slot * max_blocks + q.first - 1;
    const int32_t old = *tail;
    const int32_t nb = ring[(s_pos[tid] - 1) % P];
    if (atomicSub(&rc[old], 1) <= 1) hdr->status = KV_ERR_INTERNAL;
    rc[nb] = 1;
    *tail = nb;
    s_left[tid] = old;
    cow_pairs[tid] = make_int2(old, nb);
  }
  __threadfence_block();
  __syncthreads();
  // the host appends into a partial tail it holds alone; another table
  // referencing it would see the append's tokens.  Copies that leave it later in
  // the order of requests do not count.
  if (req && a.req[tid].cow <= 0 && a.req[tid].partial > 0) {
    const int32_t t = tables[(int64_t)a.req[tid].slot * max_blocks + a.req[tid].first - 1];
    int n = __hip_atomic_load(&rc[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (any_cow)
      for (int r = tid + 1; r < a.n_req; ++r) n += s_left[r] == t;
    if (n != 1) hdr->status = KV_ERR_INTERNAL;
  }
  for (int r = wave; r < a.n_req; r += kAllocThreads / 64) {
    int32_t* trow = tables + (int64_t)a.req[r].slot * max_blocks + a.req[r].first;
    for (int i = lane; i < a.req[r].count; i += 64) {
      const int32_t id = ring[(s_pos[r] + i) % P];
      trow[i] = id;
      rc[id] = 1;
    }
  }
}

__global__ void k_fork(DevHeader* hdr, int32_t* tables, int32_t max_blocks, int32_t* rc,
                       ForkArgs a) {
  if (hdr->status) return;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= a.nblocks) return;
  const int32_t b = tables[(int64_t)a.parent * max_blocks + j];
  rc[b] += a.k;  // ids within one table are distinct: no two threads share b
  for (int c = 0; c < a.k; ++c) tables[(int64_t)a.child[c] * max_blocks + j] = b;
}

// Exclusive prefix count of `flag` over the workgroup; returns the total.
__device__ inline int block_scan(int flag, int* excl, int* wave_tot) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const uint64_t m = __ballot(flag);
  const uint64_t below = lane ? (m & ((~0ull) >> (64 - lane))) : 0ull;
  const int in_wave = __popcll(below);
  if (lane == 0) wave_tot[wave] = __popcll(m);
  __syncthreads();
  int base = 0, total = 0;
  const int nw = blockDim.x >> 6;
  for (int w = 0; w < nw; ++w) {
    if (w < wave) base += wave_tot[w];
    total += wave_tot[w];
  }
  *excl = base + in_wave;
  __syncthreads();
  return total;
}

// cand: pairs (slot, n_blocks) in release order.  max_alloc < 0 releases all.
// truncate != 0: a candidate gives up only the blocks from its first unshared
// one (refcount 1) on, and kept[c] receives the number of leading blocks it
// keeps (0: released whole; n_blocks: nothing to give up, untouched).
// hdr->n_evicted = candidates visited before the budget was met.
__global__ void __launch_bounds__(kReleaseThreads)
k_release(DevHeader* hdr, int32_t* ring, int32_t* rc, const int32_t* tables,
          int32_t max_blocks, int32_t P, const int32_t* cand, int32_t n_cand,
          int64_t max_alloc, int64_t head, int64_t tail, int32_t truncate, int32_t* kept) {
  __shared__ int ok;
  __shared__ int first_own;
  __shared__ int wave_tot[kReleaseThreads / 64];
  if (threadIdx.x == 0) ok = hdr->status == 0 && hdr->head == head && hdr->tail == tail;
  __syncthreads();
  if (fail_if(hdr, !ok)) return;
  int n_ev = 0;
  for (int c = 0; c < n_cand; ++c) {
    if (max_alloc >= 0 && (int64_t)P - (tail - head) <= max_alloc) break;
    const int32_t slot = cand[2 * c];
    const int32_t nb = cand[2 * c + 1];
    const int32_t* trow = tables + (int64_t)slot * max_blocks;
    int start = 0;
    if (truncate) {
      if (threadIdx.x == 0) first_own = nb;
      __syncthreads();
      for (int j = threadIdx.x; j < nb; j += blockDim.x)
        if (rc[trow[j]] == 1) atomicMin(&first_own, j);
      __syncthreads();
      start = first_own;
      if (threadIdx.x == 0) kept[c] = start;
      __syncthreads();  // first_own is reset by the next candidate
      if (start == nb) {
        ++n_ev;
        continue;
      }
    }
    for (int j0 = start; j0 < nb; j0 += blockDim.x) {
      const int j = j0 + threadIdx.x;
      int flag = 0;
      int32_t b = -1;
      if (j < nb) {
        b = trow[j];
        const int32_t v = rc[b] - 1;
        rc[b] = v;
        flag = v == 0;
      }
      int excl;
      const int total = block_scan(flag, &excl, wave_tot);
      if (flag) ring[(tail + excl) % P] = b;
      tail += total;
    }
    ++n_ev;
  }
  if (threadIdx.x == 0) {
    hdr->tail = tail;
    hdr->n_evicted = n_ev;
  }
}

__global__ void __launch_bounds__(kMetaThreads)
k_compose_meta(DevHeader* hdr, int32_t* ring, int32_t* rc, int32_t* tables,
               int32_t max_blocks, int32_t P, int32_t B, int64_t head, int32_t ncopy,
               ComposeArgs a) {
  __shared__ int ok;
  if (threadIdx.x == 0) ok = hdr->status == 0 && hdr->head == head && hdr->tail - head >= ncopy;
  __syncthreads();
  if (fail_if(hdr, !ok)) return;
  int32_t* dst = tables + (int64_t)a.new_slot * max_blocks;
  for (int b = threadIdx.x; b < a.n_dest_blocks; b += blockDim.x) {
    int before = 0, seg = -1;
    for (int i = 0; i < a.nseg; ++i) {
      const int lo = a.seg[i].alias_b0, hi = a.seg[i].alias_b1;
      if (b >= lo && b < hi) seg = i;
      const int c = min(b, hi) - lo;
      before += c > 0 ? c : 0;
    }
    int32_t id;
    if (seg >= 0) {
      const SegDesc& sd = a.seg[seg];
      id = tables[(int64_t)sd.slot * max_blocks + (b - sd.off / B)];
      rc[id] += 1;  // distinct positions -> distinct source blocks
    } else {
      id = ring[(head + (b - before)) % P];
      rc[id] = 1;
    }
    dst[b] = id;
  }
  if (threadIdx.x == 0) hdr->head = head + ncopy;
}

}  // namespace

hipError_t launch_alloc(DevHeader* hdr, int32_t* ring, int32_t* rc, int32_t* tables,
                        int32_t max_blocks, int32_t P, int64_t head, const AllocArgs& a,
                        int2* cow_pairs, hipStream_t s) {
  k_alloc<<<1, kAllocThreads, 0, s>>>(hdr, ring, rc, tables, max_blocks, P, head, a, cow_pairs);
  return hipGetLastError();
}

hipError_t launch_fork(DevHeader* hdr, int32_t* tables, int32_t max_blocks, int32_t* rc,
                       const ForkArgs& a, hipStream_t s) {
  if (a.nblocks <= 0) return hipSuccess;
  const int grid = (a.nblocks + kMetaThreads - 1) / kMetaThreads;
  k_fork<<<grid, kMetaThreads, 0, s>>>(hdr, tables, max_blocks, rc, a);
  return hipGetLastError();
}

hipError_t launch_release(DevHeader* hdr, int32_t* ring, int32_t* rc, const int32_t* tables,
                          int32_t max_blocks, int32_t P, const int32_t* cand, int32_t n_cand,
                          int32_t most, int64_t max_alloc, int64_t head, int64_t tail,
                          int32_t truncate, int32_t* kept, hipStream_t s) {
  k_release<<<1, most > 768 ? kReleaseThreads : kMetaThreads, 0, s>>>(hdr, ring, rc, tables, max_blocks, P, cand, n_cand,
                                       max_alloc, head, tail, truncate, kept);
  return hipGetLastError();
}

hipError_t launch_compose_meta(DevHeader* hdr, int32_t* ring, int32_t* rc, int32_t* tables,
                               int32_t max_blocks, int32_t P, int32_t B, int64_t head,
                               int32_t ncopy, const ComposeArgs& a, hipStream_t s) {
  k_compose_meta<<<1, kMetaThreads, 0, s>>>(hdr, ring, rc, tables, max_blocks, P, B, head,
                                            ncopy, a);
  return hipGetLastError();
}

}  // namespace kvs
