// Dependence inference for implicitly parallel graphs (device side).
//
// Section 2 and Section 5 of the paper: tasks declare the data they access,
// and the runtime discovers the dependences so that the parallel execution
// equals sequential program order.  The rule applied here: tasks j < k
// conflict iff an interval of j and an interval of k overlap and at least one
// of the two is read-write; every conflicting pair becomes an edge j -> k
// (no transitive reduction, which Section 5 names as the kind of non-linear
// optimisation a compiler may avoid).
//
// Device pipeline (all on the caller's stream).  The index space is cut into
// buckets of width 2^shift; an interval has one entry, clipped to the bucket,
// in every bucket it overlaps, and a bucket keeps its writers (read-write
// intervals) and its readers in two lists:
//   1. check        : input checks and the length of the intervals by power of
//                     two (the host picks the bucket width from it);
//   2. count, scan  : list sizes (device atomics) and offsets;
//   3. entries      : entries written into their lists, in any order;
//   4. rank         : every entry counts the earlier tasks of its bucket's two
//                     lists: that is its place in task order, and the place in
//                     either list from which on its own task's successors are;
//   5. row count    : one wavefront per task tests those tails and collects the
//                     conflicting tasks in a bitmap in LDS (so a pair found
//                     twice counts once, and the row comes out ascending);
//   6. scan         : exclusive scan of row sizes -> row_ptr;
//   7. row fill     : as 5, and the bitmap is written out as the row.
// Two conflicting intervals share a bucket that holds part of their
// intersection, and there their clipped entries intersect.
//
// Where an entry list does not fit the scratch array of the allocation-free
// entry point, or a bucket is wider than 32-bit offsets, an older pipeline of
// less memory runs instead (tables of interval indices, and rows sorted at the
// end); see infer_core.
#include "taskgraph.h"
#include "tg_buckets.h"
#include "tg_internal.h"

#include <algorithm>
#include <cstring>
#include <mutex>
#include <vector>

namespace tg {

struct alignas(16) IvDev {
  uint64_t lo, hi;
  uint32_t task, priv;
};

// Empty intervals share no element and never conflict.
__device__ __forceinline__ bool iv_conflict(const IvDev& a, const IvDev& b) {
  return a.lo < a.hi && b.lo < b.hi && a.lo < b.hi && b.lo < a.hi && (a.priv == 2u || b.priv == 2u);
}

__global__ void k_bucket_count(const IvDev* iv, uint32_t M, uint32_t shift, uint32_t* bcnt) {
  const uint32_t a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= M) return;
  const IvDev x = iv[a];
  if (x.lo >= x.hi) return;
  for (uint64_t b = x.lo >> shift; b <= (x.hi - 1) >> shift; ++b) atomicAdd(bcnt + b, 1u);
}

// bent holds nent entries (the total of the scanned bucket counts).
__global__ void k_bucket_fill(const IvDev* iv, uint32_t M, uint32_t shift, const uint64_t* bptr, uint32_t* bfill,
                              uint32_t* bent, uint64_t nent) {
  const uint32_t a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= M) return;
  const IvDev x = iv[a];
  if (x.lo >= x.hi) return;
  for (uint64_t b = x.lo >> shift; b <= (x.hi - 1) >> shift; ++b) {
    const uint32_t slot = atomicAdd(bfill + b, 1u);
    const uint64_t pos = bptr[b] + slot;
    if (pos < nent) bent[pos] = a;
  }
}

// True iff (a, b) is the lexicographically first conflicting interval pair
// of tasks (j, k); a ranges over j's intervals, b over k's.
__device__ __forceinline__ bool first_pair(const IvDev* iv, const uint64_t* req_ptr, uint32_t j, uint32_t k,
                                           uint64_t a, uint64_t b) {
  const uint64_t kb = req_ptr[k], ke = req_ptr[k + 1];
  for (uint64_t a2 = req_ptr[j]; a2 <= a; ++a2) {
    const IvDev x = iv[a2];
    const uint64_t bend = (a2 == a) ? b : ke;
    for (uint64_t b2 = kb; b2 < bend; ++b2)
      if (iv_conflict(x, iv[b2])) return false;
  }
  return true;
}

// Successor scan of row j; FILL = false counts, FILL = true writes col.
template <bool FILL>
__global__ __launch_bounds__(256) void k_rows(const IvDev* iv, const uint64_t* req_ptr, uint32_t N, uint32_t shift,
                                              const uint64_t* bptr, const uint32_t* bent, uint32_t* rowcnt,
                                              const uint64_t* row_ptr, uint32_t* col) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t j = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (j >= N) return;
  uint32_t count = 0;
  uint64_t out = FILL ? row_ptr[j] : 0;
  for (uint64_t a = req_ptr[j]; a < req_ptr[j + 1]; ++a) {
    const IvDev x = iv[a];
    if (x.lo >= x.hi) continue;
    for (uint64_t B = x.lo >> shift; B <= (x.hi - 1) >> shift; ++B) {
      const uint64_t eb = bptr[B], ee = bptr[B + 1];
      for (uint64_t e0 = eb; e0 < ee; e0 += 64) {
        bool hit = false;
        uint32_t k = 0;
        if (e0 + lane < ee) {
          const uint32_t bi = bent[e0 + lane];
          const IvDev y = iv[bi];
          k = y.task;
          if (k > j && iv_conflict(x, y) && (((x.lo > y.lo) ? x.lo : y.lo) >> shift) == B)
            hit = first_pair(iv, req_ptr, j, k, a, bi);
        }
        const uint64_t m = __ballot(hit);
        if (FILL && hit) {
          const uint32_t before = __popcll(m & ((1ull << lane) - 1ull));
          col[out + before] = k;
        }
        const uint32_t c = (uint32_t)__popcll(m);
        count += c;
        out += c;
      }
    }
  }
  if (!FILL && lane == 0) rowcnt[j] = count;
}

// Interval table of a checked list, one thread per task: task k's requirements
// rq[req_ptr[k] .. req_ptr[k+1]) become IvDev entries tagged with k.
__global__ __launch_bounds__(256) void k_make_iv(const tg_region_req* rq, const uint64_t* req_ptr, uint32_t N,
                                                 IvDev* iv) {
  const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= N) return;
  for (uint64_t a = req_ptr[k]; a < req_ptr[k + 1]; ++a) {
    const tg_region_req q = rq[a];
    IvDev x;
    x.lo = q.lo;
    x.hi = q.hi;
    x.task = k;
    x.priv = q.priv;
    iv[a] = x;
  }
}

// ---------------------------------------------------------------- scan

// Exclusive scan of u32 counts into u64 offsets (out has n+1 entries).
__global__ __launch_bounds__(256) void k_scan_block(const uint32_t* in, uint64_t n, uint64_t* out, uint64_t* bsum) {
  __shared__ uint64_t s[256];
  const uint64_t base = (uint64_t)blockIdx.x * 1024;
  uint64_t v[4], t = 0;
  for (int i = 0; i < 4; ++i) {
    const uint64_t idx = base + threadIdx.x * 4 + i;
    v[i] = idx < n ? in[idx] : 0;
    t += v[i];
  }
  s[threadIdx.x] = t;
  __syncthreads();
  for (uint32_t o = 1; o < 256; o <<= 1) {
    const uint64_t add = threadIdx.x >= o ? s[threadIdx.x - o] : 0;
    __syncthreads();
    s[threadIdx.x] += add;
    __syncthreads();
  }
  uint64_t run = s[threadIdx.x] - t;
  for (int i = 0; i < 4; ++i) {
    const uint64_t idx = base + threadIdx.x * 4 + i;
    if (idx < n) out[idx] = run;
    run += v[i];
  }
  if (threadIdx.x == 255) bsum[blockIdx.x] = s[255];
}

__global__ __launch_bounds__(256) void k_scan_u64_block(uint64_t* data, uint64_t n, uint64_t* bsum) {
  __shared__ uint64_t s[256];
  const uint64_t base = (uint64_t)blockIdx.x * 1024;
  uint64_t v[4], t = 0;
  for (int i = 0; i < 4; ++i) {
    const uint64_t idx = base + threadIdx.x * 4 + i;
    v[i] = idx < n ? data[idx] : 0;
    t += v[i];
  }
  s[threadIdx.x] = t;
  __syncthreads();
  for (uint32_t o = 1; o < 256; o <<= 1) {
    const uint64_t add = threadIdx.x >= o ? s[threadIdx.x - o] : 0;
    __syncthreads();
    s[threadIdx.x] += add;
    __syncthreads();
  }
  uint64_t run = s[threadIdx.x] - t;
  for (int i = 0; i < 4; ++i) {
    const uint64_t idx = base + threadIdx.x * 4 + i;
    if (idx < n) data[idx] = run;
    run += v[i];
  }
  if (threadIdx.x == 255) bsum[blockIdx.x] = s[255];
}

__global__ void k_scan_add(uint64_t* out, uint64_t n, const uint64_t* boff) {
  const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < n) out[idx] += boff[idx / 1024];
}

__global__ void k_scan_total(uint64_t* out, uint64_t n, const uint32_t* in) {
  // out[n] = out[n-1] + in[n-1]
  if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = n ? out[n - 1] + in[n - 1] : 0;
}

__device__ __forceinline__ uint32_t rdlane(uint32_t v, uint32_t l) { return __builtin_amdgcn_readlane(v, l); }

// Inclusive sum over the lanes up to this one (all 64 active), with DPP: four
// shifted additions inside each row of 16 lanes, then the sums of the rows
// before, broadcast.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);  // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast:15, rows 1 and 3
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);  // row_bcast:31, rows 2 and 3
  return v;
}

// ------------------------------------------- entries sorted by bucket and task

// Summary of a requirement list (u64 words): error bits (1 = row pointers that
// do not run from 0 up to the interval count without decreasing, 2 = an
// interval with lo > hi or beyond the index space, 4 = an unknown privilege, 8
// = a read-write interval overlapping another interval of its own task), total
// length of the non-empty intervals, their number in each length class
// [2^c, 2^(c+1)); and the count of finished blocks.
constexpr uint32_t kSumErr = 0, kSumLen = 1, kSumClass = 2, kSumWords = 66, kSumTicket = 66, kSumAlloc = 67;

__device__ __forceinline__ bool overlaps_own(const tg_region_req& q, const tg_region_req& r) {
  return (q.priv == TG_RW || r.priv == TG_RW) && q.lo < q.hi && r.lo < r.hi && q.lo < r.hi && r.lo < q.hi;
}

// Four lanes work on a task in the kernels that go through the requirements:
// lane `sub` takes requirements sub, sub + 4, ...  Each is a chain of dependent
// round trips (row pointers, requirement, list counter, entry), and few tasks
// have more than four, so this shortens the chain to one requirement.
constexpr uint32_t kSub = 4;
// Threads of a block in those of them that end in atomics on one address
// (11 ns each, one after the other): few, large blocks.
constexpr uint32_t kTaskThreads = 1024;

// Input checks and the summary.  A task of up to four requirements compares
// them across its lanes.  The block that finishes last copies the summary to
// pinned host memory.  (One thread per task, a load per pair of requirements
// and three atomics a wavefront took 31 us of the halo program of 65,536 tasks
// with three each.)
__global__ __launch_bounds__(kTaskThreads) void k_check_reqs(const tg_region_req* rq, const uint64_t* req_ptr, uint32_t N,
                                                    uint64_t M, uint64_t space, unsigned long long* sum,
                                                    uint64_t* pin) {
  __shared__ uint32_t cls[64];
  __shared__ unsigned long long len;
  __shared__ uint32_t err, last;
  const uint32_t lane = threadIdx.x & 63u, sub = threadIdx.x % kSub;
  if (threadIdx.x < 64) cls[threadIdx.x] = 0;
  if (threadIdx.x == 64) len = 0;
  if (threadIdx.x == 65) err = 0;
  __syncthreads();
  uint32_t my_err = 0;
  unsigned long long my_len = 0;
  const uint64_t stride = (uint64_t)gridDim.x * (kTaskThreads / kSub);
  for (uint64_t k0 = (uint64_t)blockIdx.x * (kTaskThreads / kSub); k0 < N; k0 += stride) {
    const uint64_t k = k0 + threadIdx.x / kSub;
    uint64_t b = 0, e = 0;
    if (k < N) {
      b = req_ptr[k];
      e = req_ptr[k + 1];
      // the rows must partition [0, M): start at 0, never decrease, end at M
      if ((k == 0 && b != 0) || (k == N - 1 && e != M)) my_err |= 1u;
      if (e < b || e > M) {
        my_err |= 1u;
        b = e = 0;
      }
    }
    // every lane stays in the loop while any has a requirement left
    for (uint64_t i = b + sub; __ballot(i < e); i += kSub) {
      tg_region_req q;
      q.lo = q.hi = 0;
      q.priv = TG_RO;
      if (i < e) q = rq[i];
      if (q.lo > q.hi || q.hi > space) my_err |= 2u;
      if (q.priv != TG_RO && q.priv != TG_RW) my_err |= 4u;
      uint32_t c = 64;
      if (q.hi > q.lo) {
        c = 63u - (uint32_t)__clzll((long long)(q.hi - q.lo));
        my_len += q.hi - q.lo;
      }
      // one LDS addition per class present in the wavefront
      for (uint64_t left = __ballot(c < 64); left;) {
        const uint32_t c0 = __builtin_amdgcn_readlane(c, (uint32_t)__builtin_ctzll(left));
        const uint64_t same = __ballot(c == c0);
        if (lane == 0) atomicAdd(&cls[c0], (uint32_t)__popcll(same));
        left &= ~same;
      }
      // the task's other requirements of this round, then those of earlier ones
#pragma unroll
      for (uint32_t o = 1; o < kSub; ++o) {
        tg_region_req r;
        r.lo = __shfl_xor(q.lo, (int)o, 64);
        r.hi = __shfl_xor(q.hi, (int)o, 64);
        r.priv = (uint32_t)__shfl_xor((int)q.priv, (int)o, 64);
        if (overlaps_own(q, r)) my_err |= 8u;
      }
      if (i < e)
        for (uint64_t j = b; j + sub < i; ++j)
          if (overlaps_own(q, rq[j])) my_err |= 8u;
    }
  }
  for (uint32_t o = 32; o; o >>= 1) my_len += __shfl_xor(my_len, o, 64);
  if (lane == 0 && my_len) atomicAdd(&len, my_len);
  if (my_err) atomicOr(&err, my_err);
  __syncthreads();
  if (threadIdx.x < 64 && cls[threadIdx.x]) atomicAdd(sum + kSumClass + threadIdx.x, (unsigned long long)cls[threadIdx.x]);
  if (threadIdx.x == 64 && len) atomicAdd(sum + kSumLen, len);
  if (threadIdx.x == 65 && err) atomicOr(sum + kSumErr, (unsigned long long)err);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // these atomics are performed at the memory side
  __syncthreads();
  if (threadIdx.x == 0)
    last = __hip_atomic_fetch_add(sum + kSumTicket, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1ull == gridDim.x;
  __syncthreads();
  if (last && pin && threadIdx.x < kSumWords) {
    const uint64_t v = __hip_atomic_load(sum + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(pin + threadIdx.x, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// List 2B holds bucket B's writers, list 2B + 1 its readers.
__device__ __forceinline__ uint32_t list_of(uint64_t bucket, uint32_t priv) {
  return (uint32_t)(2u * bucket) + (priv == TG_RW ? 0u : 1u);
}

// List sizes.
__global__ __launch_bounds__(256) void k_list_count(const tg_region_req* rq, const uint64_t* req_ptr, uint32_t N,
                                                    uint32_t shift, uint32_t* cnt) {
  const uint64_t stride = (uint64_t)gridDim.x * (256 / kSub);
  for (uint64_t k = (uint64_t)blockIdx.x * (256 / kSub) + threadIdx.x / kSub; k < N; k += stride) {
    const uint64_t e = req_ptr[k + 1];
    for (uint64_t a = req_ptr[k] + threadIdx.x % kSub; a < e; a += kSub) {
      const tg_region_req q = rq[a];
      if (q.lo >= q.hi) continue;
      for (uint64_t b = q.lo >> shift; b <= (q.hi - 1) >> shift; ++b) atomicAdd(cnt + list_of(b, q.priv), 1u);
    }
  }
}

// An entry as the rows read it: task, and the interval's part of the bucket.
struct alignas(16) Ent {
  uint32_t task, lo, hi, pad;
};
// The same entry as its own task reads it: that part, and the bucket's writers
// and (for a read-write interval) readers whose tasks follow this one.
struct alignas(8) Own {
  uint32_t lo, hi, wpos, wlen, rpos, rlen;
};

struct EntTables {
  const uint32_t* lptr;  // list offsets, 2 x buckets + 1
  uint32_t* cnt;         // list sizes; counted down as the entries are placed
  uint32_t* utask;       // entries in the order they were placed: task ...
  uint32_t* uown;        // ... and index among the tasks' own entries
  Ent* ent;              // entries of every list, ascending in task
  Own* own;              // entries task by task: own[eoff[k] .. + ecnt[k])
  uint32_t *eoff, *ecnt;
  uint32_t nent;         // capacity of the entry arrays
};

// Entries into their lists, each list in any order.  A block reserves the
// range of its tasks' own entries with one atomic.
__global__ __launch_bounds__(kTaskThreads) void k_entries(const tg_region_req* rq, const uint64_t* req_ptr, uint32_t N,
                                                 uint32_t shift, EntTables T, unsigned long long* next) {
  __shared__ uint32_t wsum[kTaskThreads / 64];
  __shared__ uint32_t base;
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, sub = threadIdx.x % kSub;
  const uint64_t stride = (uint64_t)gridDim.x * (kTaskThreads / kSub);
  for (uint64_t k0 = (uint64_t)blockIdx.x * (kTaskThreads / kSub); k0 < N; k0 += stride) {
    const uint64_t k = k0 + threadIdx.x / kSub;
    uint64_t b = 0, e = 0;
    uint32_t n = 0;
    if (k < N) {
      b = req_ptr[k] + sub;
      e = req_ptr[k + 1];
      for (uint64_t a = b; a < e; a += kSub)
        if (rq[a].lo < rq[a].hi) n += (uint32_t)(((rq[a].hi - 1) >> shift) - (rq[a].lo >> shift) + 1);
    }
    const uint32_t incl = wave_scan(n);
    if (lane == 63) wsum[wave] = incl;
    uint32_t group = n;  // entries of the task
    group += __shfl_xor(group, 1, 64);
    group += __shfl_xor(group, 2, 64);
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t all = 0;
      for (uint32_t w = 0; w < kTaskThreads / 64; ++w) all += wsum[w];
      base = (uint32_t)atomicAdd(next, (unsigned long long)all);
    }
    __syncthreads();
    uint32_t at = base + incl - n;
    for (uint32_t w = 0; w < wave; ++w) at += wsum[w];
    if (k < N) {
      if (sub == 0) {
        T.eoff[k] = at;
        T.ecnt[k] = group;
      }
      for (uint64_t a = b; a < e; a += kSub) {
        const tg_region_req q = rq[a];
        if (q.lo >= q.hi) continue;
        for (uint64_t B = q.lo >> shift; B <= (q.hi - 1) >> shift; ++B, ++at) {
          const uint64_t start = B << shift;
          const uint32_t h = list_of(B, q.priv);
          const uint32_t u = T.lptr[h] + atomicSub(T.cnt + h, 1u) - 1u;
          if (at >= T.nent || u >= T.nent) continue;  // (the counts say it cannot be)
          T.utask[u] = (uint32_t)k;
          T.uown[u] = at;
          Own o;
          o.lo = (uint32_t)((q.lo > start ? q.lo : start) - start);
          // below 2^32: a bucket is at most 2^31 wide
          o.hi = (uint32_t)((q.hi - start) >> shift ? (1ull << shift) : q.hi - start);
          o.wpos = h;  // the list, until k_rank has read it
          o.wlen = o.rpos = o.rlen = 0;
          T.own[at] = o;
        }
      }
    }
    __syncthreads();
  }
}
static_assert(kSub == 4, "a task's entries are summed over four lanes");

// Tasks of list [b, e) below t, and not above t; ties (several intervals of
// one task in one bucket) below `u` by index.
__device__ __forceinline__ void count_tasks(const uint32_t* task, uint32_t b, uint32_t e, uint32_t t, uint32_t u,
                                            uint32_t& below, uint32_t& upto) {
  constexpr uint32_t kAhead = 16;  // loads in flight
  below = upto = 0;
  for (uint32_t i = b; i < e; i += kAhead) {
    uint32_t v[kAhead];
#pragma unroll
    for (uint32_t x = 0; x < kAhead; ++x) v[x] = i + x < e ? task[i + x] : 0xFFFFFFFFu;
#pragma unroll
    for (uint32_t x = 0; x < kAhead; ++x) {
      upto += v[x] <= t;
      below += v[x] < t || (v[x] == t && i + x < u);
    }
  }
}

// Every entry's place (one thread per placed entry; the lanes of a wavefront
// read the same list, so its loads are broadcasts).  Work is the square of a
// list's length, spread over the chip; with the about 190 entries a bucket of
// the halo program it is the latency of sixteen loads at a time (25 us).
__global__ __launch_bounds__(256) void k_rank(EntTables T, uint64_t nlists) {
  const uint32_t total = T.lptr[nlists] < T.nent ? T.lptr[nlists] : T.nent;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; u < total; u += stride) {
    const uint32_t o = T.uown[u], t = T.utask[u];
    Own w = T.own[o];
    const uint32_t h = w.wpos;
    const uint32_t b = T.lptr[h & ~1u], m = T.lptr[h | 1u], e = T.lptr[(h | 1u) + 1u];
    uint32_t wbelow, wupto, rbelow, rupto;
    count_tasks(T.utask, b, m, t, (uint32_t)u, wbelow, wupto);
    count_tasks(T.utask, m, e, t, (uint32_t)u, rbelow, rupto);
    w.wpos = b + wupto;
    w.wlen = m - w.wpos;
    w.rpos = m + rupto;
    w.rlen = (h & 1u) ? 0u : e - w.rpos;
    T.own[o] = w;
    Ent x;
    x.task = t;
    x.lo = w.lo;
    x.hi = w.hi;
    x.pad = 0;
    T.ent[(h & 1u) ? m + rbelow : b + wbelow] = x;
  }
}

// ---------------------------------------------------------------- rows

// A wavefront's bitmap: 2^wsh words a lane (wsh <= 5), so 2048 << wsh tasks.
constexpr uint32_t kMaxWordShift = 5;

__device__ __forceinline__ uint32_t first_from(const Ent* ent, uint32_t b, uint32_t e, uint32_t task) {
  while (b < e) {
    const uint32_t m = b + (e - b) / 2;
    if (ent[m].task < task) b = m + 1;
    else e = m;
  }
  return b;
}

// LDS of one wavefront is written and read by different lanes: nothing moves
// across this, in the compiler or in the wavefront.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}


// Successors of every task; FILL = false counts them, FILL = true writes them.
//
// A wavefront takes one task after another.  Lane i holds the task's i-th
// entry: its part of the bucket and the tails of the bucket's writers and (for
// a read-write entry) readers that follow the task.  The tails are read 64
// entries at a time, up to four of these loads in flight, and a conflicting
// task sets its bit in a bitmap of the tasks from the next one on (at most
// 65,536: a program of more takes several such windows, the empty ones
// skipped).  A summary word per lane says which of its bitmap words hold
// anything, so the row is read back from, and the bitmap cleared at, those
// words alone.
//
// Bound by latency: entry range, entries, tails are three dependent round
// trips a row, so the ranges are fetched two rows ahead and the entries one.
// LDS: 8 KB a wavefront for 65,536 tasks, four blocks a CU; a smaller program
// gets smaller bitmaps and up to twice the wavefronts.  Measured: 43 us to
// count and 51 us to write the 6.25 million edges of the halo program (0.26 ms
// each, and 0.38 ms for a sort, when a wavefront tested every entry of the
// buckets through an index table and rows were sorted afterwards); 26 and 29 us
// for 0.70 million edges of 30,000 tasks with four intervals (0.13, 0.13 and
// 0.10 ms).
template <bool FILL>
__global__ __launch_bounds__(256) void k_rows_sorted(EntTables T, uint32_t N, uint32_t wsh, uint32_t* rowcnt,
                                                     const uint64_t* row_ptr, uint32_t* col) {
  extern __shared__ uint32_t row_lds[];
  const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t win = 2048u << wsh;
  uint32_t* const bm = row_lds + wave * ((64u << wsh) + 64u);
  uint32_t* const sm = bm + (64u << wsh);
  for (uint32_t i = lane; i < (64u << wsh); i += 64) bm[i] = 0;
  sm[lane] = 0;
  wave_lds_sync();
  const uint32_t stride = gridDim.x * 4u;
  const uint32_t first = blockIdx.x * 4u + wave;
  const Own none = {0, 0, 0, 0, 0, 0};
  // entry ranges of this row and the next, this row's first 64 entries
  uint32_t eb = 0, ne = 0, eb1 = 0, ne1 = 0;
  if (first < N) {
    eb = T.eoff[first];
    ne = T.ecnt[first];
  }
  if ((uint64_t)first + stride < N) {
    eb1 = T.eoff[first + stride];
    ne1 = T.ecnt[first + stride];
  }
  Own o0 = none;
  if (lane < ne) o0 = T.own[eb + lane];
  for (uint64_t j0 = first; j0 < N; j0 += stride) {
    const uint32_t j = (uint32_t)j0;
    uint32_t eb2 = 0, ne2 = 0;
    if (j0 + 2ull * stride < N) {
      eb2 = T.eoff[j + 2 * stride];
      ne2 = T.ecnt[j + 2 * stride];
    }
    Own o1 = none;
    if (lane < ne1) o1 = T.own[eb1 + lane];
    uint32_t count = 0;
    uint64_t out = FILL ? row_ptr[j] : 0;
    uint32_t base = j + 1;
    while (base < N) {
      const bool more = N - base > win;  // tasks past this window
      uint32_t next = 0xFFFFFFFFu;       // the first task found there
      for (uint32_t c = 0; c < ne; c += 64) {
        Own o = o0;
        if (c) {
          o = none;
          if (c + lane < ne) o = T.own[eb + c + lane];
        }
        if (base != j + 1u) {
          const uint32_t w = first_from(T.ent, o.wpos, o.wpos + o.wlen, base), r = first_from(T.ent, o.rpos, o.rpos + o.rlen, base);
          o.wlen -= w - o.wpos;
          o.rlen -= r - o.rpos;
          o.wpos = w;
          o.rpos = r;
        }
        if (more) {
          const uint32_t w = first_from(T.ent, o.wpos, o.wpos + o.wlen, base + win), r = first_from(T.ent, o.rpos, o.rpos + o.rlen, base + win);
          if (w < o.wpos + o.wlen) next = min(next, T.ent[w].task);
          if (r < o.rpos + o.rlen) next = min(next, T.ent[r].task);
          o.wlen = w - o.wpos;
          o.rlen = r - o.rpos;
        }
        uint64_t todo = __ballot(o.wlen + o.rlen != 0u);
        uint32_t i0 = 0;
        while (todo) {
          Ent x[4];
          uint32_t xlo[4], xhi[4];
          bool ok[4];
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            ok[s] = false;
            xlo[s] = xhi[s] = 0;
            if (todo) {
              const uint32_t l = (uint32_t)__builtin_ctzll(todo);
              const uint32_t wl = rdlane(o.wlen, l), len = wl + rdlane(o.rlen, l);
              const uint32_t wp = rdlane(o.wpos, l), rp = rdlane(o.rpos, l);
              const uint32_t i = i0 + lane;
              ok[s] = i < len;
              if (ok[s]) x[s] = T.ent[i < wl ? wp + i : rp + (i - wl)];
              xlo[s] = rdlane(o.lo, l);
              xhi[s] = rdlane(o.hi, l);
              i0 += 64;
              if (i0 >= len) {
                i0 = 0;
                todo &= todo - 1;
              }
            }
          }
#pragma unroll
          for (int s = 0; s < 4; ++s)
            if (ok[s] && x[s].lo < xhi[s] && xlo[s] < x[s].hi) {
              // bit d of the window: word d / 32 of lane d / 32 >> wsh, the
              // lanes' words side by side so that they lie in different banks
              const uint32_t d = x[s].task - base, w = d >> 5, l = w >> wsh, k = w & ((1u << wsh) - 1u);
              __hip_atomic_fetch_or(bm + k * 64u + l, 1u << (d & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
              __hip_atomic_fetch_or(sm + l, 1u << k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            }
        }
      }
      wave_lds_sync();
      const uint32_t words = sm[lane];
      sm[lane] = 0;
      uint32_t mine = 0;
      for (uint32_t t = words; t; t &= t - 1) {
        uint32_t* p = bm + (uint32_t)__builtin_ctz(t) * 64u + lane;
        mine += (uint32_t)__popc(*p);
        if (!FILL) *p = 0;
      }
      if (FILL) {
        const uint32_t incl = wave_scan(mine);
        uint64_t at = out + (incl - mine);
        for (uint32_t t = words; t; t &= t - 1) {
          const uint32_t k = (uint32_t)__builtin_ctz(t);
          uint32_t* p = bm + k * 64u + lane;
          const uint32_t task0 = base + ((lane << wsh) + k) * 32u;
          for (uint32_t v = *p; v; v &= v - 1) col[at++] = task0 + (uint32_t)__builtin_ctz(v);
          *p = 0;
        }
        out += rdlane(incl, 63);
      } else {
        count += mine;
      }
      wave_lds_sync();
      if (!more) break;
      for (uint32_t k = 32; k; k >>= 1) next = min(next, (uint32_t)__shfl_xor(next, k, 64));
      base = rdlane(next, 0);
      if (base == 0xFFFFFFFFu) break;
    }
    if (!FILL) {
      const uint32_t sum = wave_scan(count);
      if (lane == 63) rowcnt[j] = sum;
    }
    eb = eb1;
    ne = ne1;
    eb1 = eb2;
    ne1 = ne2;
    o0 = o1;
  }
}

// Sum of each tile of `tile` counts.
__global__ __launch_bounds__(256) void k_tile_sums(const uint32_t* in, uint64_t n, uint64_t tile, uint64_t* sums) {
  __shared__ uint64_t s[4];
  const uint64_t b = blockIdx.x * tile, e = b + tile < n ? b + tile : n;
  uint64_t v = 0;
  for (uint64_t i = b + threadIdx.x; i < e; i += 256) v += in[i];
  for (uint32_t o = 32; o; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63u) == 0) s[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) sums[blockIdx.x] = s[0] + s[1] + s[2] + s[3];
}

// out[0..n] = exclusive scan of in[0..n), out[n] the total, which also goes to
// *pin (pinned host memory) if there is one.  A block adds up the sums of the
// tiles before its own (at most 2048, so no block waits for another), then
// goes through its tile 1024 counts at a time.
template <class Out>
__global__ __launch_bounds__(256) void k_tile_scan(const uint32_t* in, uint64_t n, uint64_t tile, const uint64_t* sums,
                                                   Out* out, uint64_t* pin) {
  __shared__ uint64_t s[4];
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  uint64_t v = 0;
  for (uint32_t i = threadIdx.x; i < blockIdx.x; i += 256) v += sums[i];
  for (uint32_t o = 32; o; o >>= 1) v += __shfl_xor(v, o, 64);
  if (lane == 0) s[wave] = v;
  __syncthreads();
  uint64_t run = s[0] + s[1] + s[2] + s[3];
  const uint64_t b = blockIdx.x * tile, e = b + tile < n ? b + tile : n;
  for (uint64_t c = b; c < e; c += 1024) {
    const uint64_t i0 = c + threadIdx.x * 4u;
    uint32_t x[4];
    uint64_t mine = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i] = i0 + i < e ? in[i0 + i] : 0u;
      mine += x[i];
    }
    uint64_t incl = mine;
    for (uint32_t o = 1; o < 64; o <<= 1) {
      const uint64_t y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    __syncthreads();  // everybody has read the sums of the last round
    if (lane == 63) s[wave] = incl;
    __syncthreads();
    uint64_t at = run + incl - mine;
    for (uint32_t w = 0; w < 4; ++w) {
      if (w < wave) at += s[w];
      run += s[w];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i0 + i < e) out[i0 + i] = (Out)at;
      at += x[i];
    }
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    out[n] = (Out)run;
    if (pin) __hip_atomic_store(pin, run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

constexpr uint64_t kMaxTiles = 2048;

// Scan of n >= 1 counts in at most two launches; sums: kMaxTiles words.
template <class Out>
static hipError_t tile_scan(const uint32_t* in, uint64_t n, Out* out, uint64_t* sums, uint64_t* pin, hipStream_t st) {
  uint64_t tile = ((n + kMaxTiles - 1) / kMaxTiles + 1023) & ~1023ull;
  if (n <= 4096) tile = 4096;  // one block, one launch
  const uint32_t nt = (uint32_t)((n + tile - 1) / tile);
  hipError_t e = hipSuccess;
  if (nt > 1) {
    hipLaunchKernelGGL(k_tile_sums, dim3(nt), dim3(256), 0, st, in, n, tile, sums);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_tile_scan<Out>, dim3(nt), dim3(256), 0, st, in, n, tile, sums, out, pin);
  return hipGetLastError();
}

// Device memory of one inference: carved in order from a fixed region (one of
// the scratch arrays), or allocated and freed when the workspace goes away.  In
// the allocation-free entry point a request that does not fit the region fails
// and names the array.
struct Workspace {
  uint8_t* base = nullptr;  // fixed region; null: allocate
  size_t cap = 0, used = 0;
  bool spill = true;        // allocate what does not fit
  std::vector<void*> owned;
  const char* missing = nullptr;  // array that did not fit
  Workspace() = default;
  Workspace(const Workspace&) = delete;
  Workspace& operator=(const Workspace&) = delete;
  ~Workspace() {
    for (void* p : owned) (void)hipFree(p);
  }
  hipError_t get(size_t bytes, const char* name, void** out) {
    bytes = bytes ? (bytes + 255) & ~(size_t)255 : 256;
    if (bytes <= cap - used) {
      *out = base + used;
      used += bytes;
      return hipSuccess;
    }
    if (!spill) {
      missing = name;
      return hipErrorOutOfMemory;
    }
    const hipError_t e = hipMalloc(out, bytes);
    if (e == hipSuccess) owned.push_back(*out);
    return e;
  }
  // Gives back what was taken since the region was at `used0` with `owned0`
  // allocations; the device must have finished with it.
  void rewind(size_t used0, size_t owned0) {
    used = used0;
    missing = nullptr;
    for (; owned.size() > owned0; owned.pop_back()) (void)hipFree(owned.back());
  }
};

__global__ void k_fill_u32(uint32_t* p, uint64_t n, uint32_t v) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

// Clears device words with a kernel (callers may record the work into a HIP
// graph, where memset nodes are avoided).
static hipError_t fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t st) {
  if (n == 0) return hipSuccess;
  uint64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_fill_u32, dim3((uint32_t)blocks), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

// In-place exclusive scan of u64 (used recursively for block sums).
static hipError_t scan_u64_inplace(uint64_t* data, uint64_t n, Workspace& ws, hipStream_t st) {
  if (n <= 1) return n == 1 ? fill_u32((uint32_t*)data, 2, 0, st) : hipSuccess;
  const uint64_t nb = (n + 1023) / 1024;
  void* bs = nullptr;
  hipError_t e = ws.get(nb * 8, "scan partial sums", &bs);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_scan_u64_block, dim3((uint32_t)nb), dim3(256), 0, st, data, n, (uint64_t*)bs);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (nb > 1) {
    if ((e = scan_u64_inplace((uint64_t*)bs, nb, ws, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_scan_add, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, st, data, n, (const uint64_t*)bs);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

// out[0..n] = exclusive scan of in[0..n) with out[n] = total (stream-ordered).
static hipError_t scan_counts(const uint32_t* in, uint64_t n, uint64_t* out, Workspace& ws, hipStream_t st) {
  if (n == 0) return fill_u32((uint32_t*)out, 2, 0, st);
  const uint64_t nb = (n + 1023) / 1024;
  void* bs = nullptr;
  hipError_t e = ws.get(nb * 8, "scan partial sums", &bs);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_scan_block, dim3((uint32_t)nb), dim3(256), 0, st, in, n, out, (uint64_t*)bs);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (nb > 1) {
    if ((e = scan_u64_inplace((uint64_t*)bs, nb, ws, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_scan_add, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, st, out, n, (const uint64_t*)bs);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_scan_total, dim3(1), dim3(1), 0, st, out, n, in);
  return hipGetLastError();
}

// ------------------------------------------------------------- row sort

constexpr uint32_t kSortLds = 8192;  // words staged in LDS per row

__device__ __forceinline__ void cswap_lds(uint32_t* a, uint32_t i, uint32_t j) {
  const uint32_t x = a[i], y = a[j];
  if (y < x) {
    a[i] = y;
    a[j] = x;
  }
}

// Ascending bitonic network over a virtual array padded to a power of two
// with +infinity; every comparator puts the minimum at the lower index, so
// comparators touching the padding are no-ops and are skipped.
__global__ __launch_bounds__(1024) void k_sort_rows(const uint64_t* row_ptr, uint32_t N, uint32_t* col) {
  __shared__ uint32_t s[kSortLds];
  const uint32_t row = blockIdx.x;
  if (row >= N) return;
  const uint64_t b = row_ptr[row];
  const uint32_t L = (uint32_t)(row_ptr[row + 1] - b);
  if (L < 2) return;
  uint32_t P = 1;
  while (P < L) P <<= 1;
  if (L <= kSortLds) {
    for (uint32_t i = threadIdx.x; i < L; i += blockDim.x) s[i] = col[b + i];
    __syncthreads();
    for (uint32_t k = 2; k <= P; k <<= 1) {
      // flip step
      for (uint32_t i = threadIdx.x; i < P / 2; i += blockDim.x) {
        const uint32_t blk = i / (k / 2), off = i % (k / 2);
        const uint32_t lo = blk * k + off, hi = blk * k + k - 1 - off;
        if (hi < L) cswap_lds(s, lo, hi);
      }
      __syncthreads();
      for (uint32_t h = k / 4; h >= 1; h >>= 1) {
        for (uint32_t i = threadIdx.x; i < P / 2; i += blockDim.x) {
          const uint32_t blk = i / h, off = i % h;
          const uint32_t lo = blk * 2 * h + off, hi = lo + h;
          if (hi < L) cswap_lds(s, lo, hi);
        }
        __syncthreads();
      }
    }
    for (uint32_t i = threadIdx.x; i < L; i += blockDim.x) col[b + i] = s[i];
  } else {
    uint32_t* a = col + b;
    for (uint32_t k = 2; k <= P; k <<= 1) {
      for (uint32_t i = threadIdx.x; i < P / 2; i += blockDim.x) {
        const uint32_t blk = i / (k / 2), off = i % (k / 2);
        const uint32_t lo = blk * k + off, hi = blk * k + k - 1 - off;
        if (hi < L) {
          const uint32_t x = __hip_atomic_load(a + lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          const uint32_t y = __hip_atomic_load(a + hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (y < x) {
            __hip_atomic_store(a + lo, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(a + hi, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __syncthreads();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
      for (uint32_t h = k / 4; h >= 1; h >>= 1) {
        for (uint32_t i = threadIdx.x; i < P / 2; i += blockDim.x) {
          const uint32_t blk = i / h, off = i % h;
          const uint32_t lo = blk * 2 * h + off, hi = lo + h;
          if (hi < L) {
            const uint32_t x = __hip_atomic_load(a + lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t y = __hip_atomic_load(a + hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (y < x) {
              __hip_atomic_store(a + lo, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              __hip_atomic_store(a + hi, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
      }
    }
  }
}

// ------------------------------------------------------- initial array

__global__ void k_init_data(uint32_t* A, uint64_t space, uint64_t key2) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < space; e += stride) {
    uint64_t z = key2 ^ e;
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    A[e] = (uint32_t)(z ^ (z >> 31));
  }
}

}  // namespace tg

hipError_t tg_launch_init_data(uint32_t* A, uint64_t space, uint64_t key2, hipStream_t s) {
  uint64_t blocks = (space + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  if (blocks == 0) blocks = 1;
  hipLaunchKernelGGL(tg::k_init_data, dim3((uint32_t)blocks), dim3(256), 0, s, A, space, key2);
  return hipGetLastError();
}

// ------------------------------------------------------------ host driver

namespace {

using tg::IvDev;
using tg::Workspace;

size_t round256(uint64_t b) { return (size_t)((b + 255) & ~255ull); }

// Bucket width 2^shift: the power of two nearest the mean non-empty interval
// length, widened until the index space needs at most max_buckets buckets.
uint32_t choose_shift(unsigned long long total_len, unsigned long long nonempty, uint64_t space,
                      uint64_t max_buckets) {
  uint32_t shift = 0;
  if (nonempty) {
    const long double mean = (long double)total_len / (long double)nonempty;
    while (shift < 40 && (long double)(1ull << (shift + 1)) <= mean * 1.41421356L) shift++;
  }
  while (((space + (1ull << shift) - 1) >> shift) > max_buckets) shift++;
  return shift;
}

// Copies `bytes` of device memory to host memory on `st` and waits.
hipError_t read_back(void* host, const void* dev, size_t bytes, hipStream_t st) {
  const hipError_t e = hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, st);
  return e == hipSuccess ? hipStreamSynchronize(st) : e;
}

// One array of device memory that the code object defines, for the inferences
// that do not allocate.  Each device holds its own copy of the array until the
// process ends.  On the host, `scratch` names only a stand-in for the device
// symbol: its device address comes from hipGetSymbolAddress, taken once per
// device with that device current, and only that address is handed to kernels
// and copies.
constexpr size_t kScratchBytes = size_t(16) << 20;
static __device__ __align__(256) uint8_t scratch[kScratchBytes];
// A second one for the inferences that may allocate: the call that finds it
// free uses it and allocates what does not fit.  (A pair of hipMalloc and
// hipFree above 2 MiB costs 30 to 60 us, at times 600, beside 130 us of kernels
// for 30,000 tasks.)  It is not the first one, so an allocation-free call never
// waits for an inference of the other kind.
constexpr size_t kSpareBytes = size_t(32) << 20;
static __device__ __align__(256) uint8_t spare[kSpareBytes];


constexpr int kMaxDevices = 64;
constexpr uint64_t kNoallocMaxBuckets = 1ull << 18;  // bucket arrays of at most 3 MiB

struct ScratchDev {
  std::once_flag once;
  void* ptr = nullptr;
  hipError_t err = hipSuccess;
  void* spare_ptr = nullptr;
  std::mutex mu;        // one allocation-free call at a time per device in this process
  std::mutex spare_mu;  // the user of the second array
};
ScratchDev g_scratch[kMaxDevices];

// The calling thread's device's scratch array.
tg_status scratch_of_device(ScratchDev** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return tg_set_error(TG_EDEVICE, "hipGetDevice: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices)
    return tg_set_error(TG_EDEVICE, "device %d: the scratch table holds devices 0..%d", dev, kMaxDevices - 1);
  ScratchDev& sd = g_scratch[dev];
  std::call_once(sd.once, [&sd] {
    sd.err = hipGetSymbolAddress(&sd.ptr, HIP_SYMBOL(scratch));
    if (hipGetSymbolAddress(&sd.spare_ptr, HIP_SYMBOL(spare)) != hipSuccess) {
      sd.spare_ptr = nullptr;
      (void)hipGetLastError();
    }
  });
  if (sd.err != hipSuccess || !sd.ptr)
    return tg_set_error(TG_EDEVICE, "hipGetSymbolAddress of the scratch array on device %d: %s", dev,
                        hipGetErrorString(sd.err));
  *out = &sd;
  return TG_OK;
}

// The second scratch array for one inference, if nobody has it; given back
// once the inference's stream has finished with it.
class SpareUse {
 public:
  SpareUse(Workspace& ws, hipStream_t st) : st_(st) {
    ScratchDev* sd = nullptr;
    if (scratch_of_device(&sd) != TG_OK || !sd->spare_ptr || !sd->spare_mu.try_lock()) return;
    sd_ = sd;
    ws.base = (uint8_t*)sd->spare_ptr;
    ws.cap = kSpareBytes;
  }
  ~SpareUse() {
    if (!sd_) return;
    (void)hipStreamSynchronize(st_);
    sd_->spare_mu.unlock();
  }
  SpareUse(const SpareUse&) = delete;
  SpareUse& operator=(const SpareUse&) = delete;

 private:
  ScratchDev* sd_ = nullptr;
  hipStream_t st_;
};

// Pinned host words that kernels store small results into (a copy engine's
// read-back costs about 10 us more).  One block per inference in flight, kept
// for the next; a process holds as many as its allocating inferences ever ran at
// once.  An allocation-free call (make = false) uses a block that one of those
// left and makes none.  Without a block the results are copied back instead.
struct PinBlock {
  static constexpr size_t kWords = 128;  // the summary, then the edge and entry counts
  uint64_t* p = nullptr;
  explicit PinBlock(bool make) {
    Pool& pl = pool();
    std::lock_guard<std::mutex> lk(pl.mu);
    if (!pl.free.empty()) {
      p = pl.free.back();
      pl.free.pop_back();
      return;
    }
    if (!make) return;
    pl.free.reserve(pl.made + 1);  // giving a block back never allocates
    void* v = nullptr;
    // portable: the pool serves every device
    if (hipHostMalloc(&v, kWords * 8, hipHostMallocCoherent | hipHostMallocMapped | hipHostMallocPortable) == hipSuccess) {
      p = (uint64_t*)v;
      ++pl.made;
    } else {
      (void)hipGetLastError();
    }
  }
  ~PinBlock() {
    if (!p) return;
    std::lock_guard<std::mutex> lk(pool().mu);
    pool().free.push_back(p);
  }
  PinBlock(const PinBlock&) = delete;
  PinBlock& operator=(const PinBlock&) = delete;

 private:
  struct Pool {
    std::mutex mu;
    std::vector<uint64_t*> free;
    size_t made = 0;
  };
  static Pool& pool() {
    static Pool* pl = new Pool;
    return *pl;
  }
};

#define ICHK(x, what)                                                                                   \
  do {                                                                                                  \
    e = (x);                                                                                            \
    if (e != hipSuccess) {                                                                              \
      if (ws.missing)                                                                                   \
        return tg_set_error(TG_ENOMEM, "dependence inference: the %s do not fit the %zu-byte scratch array", \
                            ws.missing, ws.cap);                                                        \
      return tg_set_error(TG_EDEVICE, "dependence inference (%s): %s", what, hipGetErrorString(e));     \
    }                                                                                                   \
  } while (0)

// Whether a DAG of E edges can be returned (a caller's buffer holds col_cap).
tg_status edge_count_ok(uint64_t E, bool alloc_col, uint64_t col_cap) {
  if (E >= 0xFFFFFFFFull) return tg_set_error(TG_EINVAL, "inferred DAG has too many edges (%llu)", (unsigned long long)E);
  if (!alloc_col && E > col_cap)
    return tg_set_error(TG_ENOMEM, "inferred DAG has %llu edges, capacity %llu", (unsigned long long)E,
                        (unsigned long long)col_cap);
  return TG_OK;
}

// The edge buffer of a counted DAG (E edges), as infer_steps' contract.
tg_status edge_buffer(Workspace& ws, uint64_t E, uint32_t** col, bool alloc_col, uint64_t col_cap) {
  hipError_t e;
  const tg_status s = edge_count_ok(E, alloc_col, col_cap);
  if (s != TG_OK) return s;
  if (alloc_col) ICHK(ws.get(E * 4, "edges", (void**)col), "edge array");
  return TG_OK;
}

uint32_t task_blocks(uint64_t threads) {
  const uint64_t b = (threads + 255) / 256;
  return (uint32_t)(b > 4096 ? 4096 : b ? b : 1);
}

// Blocks of the kernels with kTaskThreads threads: one per CU at most.
uint32_t big_blocks(uint32_t N) {
  return (uint32_t)std::min<uint64_t>(((uint64_t)N * tg::kSub + tg::kTaskThreads - 1) / tg::kTaskThreads, 256);
}

// Rows from sorted entries.  *done = false (and nothing but scratch memory and
// row touched) if the entries do not fit the workspace's fixed region or, where it
// may allocate, the device's memory: the other pipeline takes a tenth of it.
tg_status infer_entries(Workspace& ws, uint32_t N, uint64_t space, const tg_region_req* rq, const uint64_t* req_ptr,
                        uint32_t shift, uint64_t nent_bound, hipStream_t st, uint64_t* pin, uint64_t* row, uint32_t** col,
                        bool alloc_col, uint64_t col_cap, uint64_t* E, bool* done) {
  *done = false;
  hipError_t e;
  const uint64_t nlists = 2 * (((space - 1) >> shift) + 1);
  const size_t used0 = ws.used, owned0 = ws.owned.size();
  auto give_up = [&] {  // everything taken here goes back, once the stream has finished with it
    (void)hipGetLastError();
    e = hipStreamSynchronize(st);
    ws.rewind(used0, owned0);
    return e == hipSuccess ? TG_OK
                           : tg_set_error(TG_EDEVICE, "dependence inference (entries): %s", hipGetErrorString(e));
  };
  // list sizes and the entry allocator are cleared together
  const size_t cnt_bytes = round256(nlists * 4), lptr_bytes = round256((nlists + 1) * 4);
  const size_t fixed = cnt_bytes + 256 + lptr_bytes + tg::kMaxTiles * 8 + 2 * round256((uint64_t)N * 4) + round256((uint64_t)N * 4);
  auto entry_bytes = [](uint64_t n) {
    return round256(n * sizeof(tg::Own)) + round256(n * sizeof(tg::Ent)) + 2 * round256(n * 4);
  };
  auto fits = [&](uint64_t n) { return fixed + entry_bytes(n) + 8192 <= ws.cap - used0; };
  // (a fixed region that does not even hold the lists: the other pipeline)
  if (!ws.spill && !fits(0)) return TG_OK;
  uint8_t* fx = nullptr;
  e = ws.get(fixed, "lists", (void**)&fx);
  if (e == hipErrorOutOfMemory) return give_up();
  ICHK(e, "lists");
  tg::EntTables T;
  T.cnt = (uint32_t*)fx;
  unsigned long long* next = (unsigned long long*)(fx + cnt_bytes);
  uint32_t* lptr = (uint32_t*)(fx + cnt_bytes + 256);
  uint64_t* sums = (uint64_t*)((uint8_t*)lptr + lptr_bytes);
  T.lptr = lptr;
  T.eoff = (uint32_t*)((uint8_t*)sums + tg::kMaxTiles * 8);
  T.ecnt = T.eoff + round256((uint64_t)N * 4) / 4;
  uint32_t* rcnt = T.ecnt + round256((uint64_t)N * 4) / 4;
  const uint32_t tb = task_blocks((uint64_t)N * tg::kSub);
  ICHK(tg::fill_u32(T.cnt, (cnt_bytes + 256) / 4, 0, st), "clear");
  hipLaunchKernelGGL(tg::k_list_count, dim3(tb), dim3(256), 0, st, rq, req_ptr, N, shift, T.cnt);
  ICHK(hipGetLastError(), "k_list_count");
  uint64_t* pin_n = pin ? pin + tg::kSumAlloc : nullptr;
  ICHK(tg::tile_scan<uint32_t>(T.cnt, nlists, lptr, sums, pin_n, st), "list scan");
  uint64_t nent = nent_bound;
  if (!fits(nent)) {
    // the bound allows two partly covered buckets per interval: ask for the
    // number itself before the entries are refused, or allocated
    if (pin) {
      ICHK(hipStreamSynchronize(st), "list scan");
      nent = __atomic_load_n(pin_n, __ATOMIC_ACQUIRE);
    } else {
      uint32_t n32 = 0;
      ICHK(read_back(&n32, lptr + nlists, 4, st), "entry count read-back");
      nent = n32;
    }
    if (!ws.spill && !fits(nent)) return give_up();
  }
  uint8_t* ex = nullptr;
  e = ws.get(entry_bytes(nent), "entries", (void**)&ex);
  if (e == hipErrorOutOfMemory) return give_up();
  ICHK(e, "entries");
  T.own = (tg::Own*)ex;
  T.ent = (tg::Ent*)(ex + round256(nent * sizeof(tg::Own)));
  T.utask = (uint32_t*)((uint8_t*)T.ent + round256(nent * sizeof(tg::Ent)));
  T.uown = T.utask + round256(nent * 4) / 4;
  T.nent = (uint32_t)nent;
  hipLaunchKernelGGL(tg::k_entries, dim3(big_blocks(N)), dim3(tg::kTaskThreads), 0, st, rq, req_ptr, N, shift, T, next);
  ICHK(hipGetLastError(), "k_entries");
  hipLaunchKernelGGL(tg::k_rank, dim3(task_blocks(nent)), dim3(256), 0, st, T, nlists);
  ICHK(hipGetLastError(), "k_rank");
  // bitmaps as large as the program needs, as many blocks as their LDS (of 160
  // KB a CU) and eight wavefronts a SIMD admit on 256 CUs
  uint32_t wsh = 0;
  while (wsh < tg::kMaxWordShift && (2048u << wsh) < N) ++wsh;
  const uint32_t lds = 4u * ((64u << wsh) + 64u) * 4u;
  const uint32_t rb = (uint32_t)std::min<uint64_t>(((uint64_t)N + 3) / 4, 256u * std::min(8u, 163840u / lds));
  hipLaunchKernelGGL(tg::k_rows_sorted<false>, dim3(rb), dim3(256), lds, st, T, N, wsh, rcnt, (const uint64_t*)nullptr,
                     (uint32_t*)nullptr);
  ICHK(hipGetLastError(), "k_rows_sorted (count)");
  uint64_t* pin_e = pin ? pin + tg::kSumAlloc + 1 : nullptr;
  ICHK(tg::tile_scan<uint64_t>(rcnt, N, row, sums, pin_e, st), "row scan");
  if (pin) {
    ICHK(hipStreamSynchronize(st), "row counts");
    *E = __atomic_load_n(pin_e, __ATOMIC_ACQUIRE);
  } else {
    ICHK(read_back(E, row + N, 8, st), "edge count read-back");
  }
  if (alloc_col && *E < 0xFFFFFFFFull) {
    e = ws.get(*E * 4, "edges", (void**)col);
    if (e == hipErrorOutOfMemory) return give_up();
    ICHK(e, "edge array");
  }
  *done = true;
  const tg_status s = edge_count_ok(*E, alloc_col, col_cap);
  if (s != TG_OK) return s;
  if (*E) {
    hipLaunchKernelGGL(tg::k_rows_sorted<true>, dim3(rb), dim3(256), lds, st, T, N, wsh, rcnt, row, *col);
    ICHK(hipGetLastError(), "k_rows_sorted (fill)");
  }
  ICHK(hipStreamSynchronize(st), "inference");
  return TG_OK;
}

// Inference proper, on device inputs, all work ordered on `st`:
//   rq[M], req_ptr[N+1] : the requirements (device);
//   row[N+1]            : receives the out-edge row pointers (device);
//   *col                : receives the successors: when alloc_col is set a
//                         buffer of the exact size is taken from the
//                         workspace, else *col (capacity col_cap) is used
//                         and a larger edge count fails with TG_ENOMEM;
//   *E                  : the edge count (set also on TG_ENOMEM);
//   pin                 : pinned words for the small results, or null.
// Returns when the DAG is complete on the device.
tg_status infer_steps(Workspace& ws, uint32_t N, uint64_t M, uint64_t space, const tg_region_req* rq,
                      const uint64_t* req_ptr, uint64_t max_buckets, hipStream_t st, uint64_t* pin, uint64_t* row,
                      uint32_t** col, bool alloc_col, uint64_t col_cap, uint64_t* E) {
  hipError_t e;
  *E = 0;
  if (M >= 0xFFFFFFFFull) return tg_set_error(TG_EINVAL, "too many region requirements");
  const uint32_t M32 = (uint32_t)M;
  const size_t used0 = ws.used;
  unsigned long long* summary = nullptr;
  ICHK(ws.get(tg::kSumAlloc * 8, "summary", (void**)&summary), "summary");
  ICHK(tg::fill_u32((uint32_t*)summary, tg::kSumAlloc * 2, 0, st), "clear");
  hipLaunchKernelGGL(tg::k_check_reqs, dim3(big_blocks(N)), dim3(tg::kTaskThreads), 0, st, rq, req_ptr, N, M,
                     space, summary, pin);
  ICHK(hipGetLastError(), "k_check_reqs");
  uint64_t sum[tg::kSumWords];
  if (pin) {
    ICHK(hipStreamSynchronize(st), "requirement check");
    for (uint32_t i = 0; i < tg::kSumWords; ++i) sum[i] = __atomic_load_n(pin + i, __ATOMIC_ACQUIRE);
  } else {
    ICHK(read_back(sum, summary, sizeof(sum), st), "summary read-back");
  }
  if (sum[tg::kSumErr]) {
    const uint32_t b = (uint32_t)sum[tg::kSumErr];
    return tg_set_error(TG_EINVAL, "region requirements: %s%s%s%s",
                        (b & 1) ? "row pointers do not run from 0 to the requirement count without decreasing; " : "",
                        (b & 2) ? "interval with lo > hi or outside the index space; " : "",
                        (b & 4) ? "unknown privilege; " : "",
                        (b & 8) ? "read-write interval overlapping another interval of its task" : "");
  }
  uint64_t nonempty = 0;
  for (int c = 0; c < 64; ++c) nonempty += sum[tg::kSumClass + c];
  if (nonempty == 0) {  // no element is declared: no edges
    ICHK(tg::fill_u32((uint32_t*)row, 2 * ((uint64_t)N + 1), 0, st), "clear");
    const tg_status s = edge_buffer(ws, 0, col, alloc_col, col_cap);
    if (s != TG_OK) return s;
    ICHK(hipStreamSynchronize(st), "inference");
    return TG_OK;
  }
  {
    // the total length, or a bound on it if it may have overflowed
    long double length = 0;
    for (int c = 0; c < 64; ++c) length += (long double)sum[tg::kSumClass + c] * 2.0L * (long double)(1ull << c);
    if (length < 1.8e19L) length = (long double)sum[tg::kSumLen];
    const uint32_t es = tg::entry_shift(sum + tg::kSumClass, nonempty, length, space, max_buckets / 2);
    // an interval of length l touches at most (l >> shift) + 2 buckets
    const long double bound = 2.0L * (long double)nonempty + length / (long double)(1ull << es);
    // 32-bit offsets inside a bucket, and 32-bit entry indices
    if (es <= 31 && bound < 4.0e9L) {
      bool done = false;
      const tg_status s = infer_entries(ws, N, space, rq, req_ptr, es, (uint64_t)bound + 1, st, pin, row, col, alloc_col,
                                        col_cap, E, &done);
      if (s != TG_OK || done) return s;
    }
  }
  // The older pipeline: 4 bytes an entry where the sorted entries take 48, so
  // requirement lists near the scratch array's limit still fit.
  ws.used = used0;  // (a fixed region: the summary has been read)
  IvDev* iv = nullptr;
  ICHK(ws.get(M * sizeof(IvDev), "intervals", (void**)&iv), "interval table");
  hipLaunchKernelGGL(tg::k_make_iv, dim3((N + 255) / 256), dim3(256), 0, st, rq, req_ptr, N, iv);
  ICHK(hipGetLastError(), "k_make_iv");
  const uint32_t shift = choose_shift(sum[tg::kSumLen], nonempty, space, max_buckets);
  const uint64_t nb = (space + (1ull << shift) - 1) >> shift;
  uint32_t* bcnt = nullptr;
  uint64_t* bptr = nullptr;
  ICHK(ws.get(nb * 4, "bucket counts", (void**)&bcnt), "bucket counts");
  ICHK(ws.get((nb + 1) * 8, "bucket offsets", (void**)&bptr), "bucket offsets");
  ICHK(tg::fill_u32(bcnt, nb, 0, st), "clear");
  if (M32) {
    hipLaunchKernelGGL(tg::k_bucket_count, dim3((M32 + 255) / 256), dim3(256), 0, st, iv, M32, shift, bcnt);
    ICHK(hipGetLastError(), "k_bucket_count");
  }
  ICHK(tg::scan_counts(bcnt, nb, bptr, ws, st), "bucket scan");
  uint64_t nent = 0;
  ICHK(read_back(&nent, bptr + nb, 8, st), "bucket total read-back");
  uint32_t* bent = nullptr;
  ICHK(ws.get(nent * 4, "bucket entries", (void**)&bent), "bucket entries");
  ICHK(tg::fill_u32(bcnt, nb, 0, st), "clear");
  if (M32) {
    hipLaunchKernelGGL(tg::k_bucket_fill, dim3((M32 + 255) / 256), dim3(256), 0, st, iv, M32, shift, bptr, bcnt, bent,
                       nent);
    ICHK(hipGetLastError(), "k_bucket_fill");
  }
  uint32_t* rcnt = nullptr;
  ICHK(ws.get((size_t)N * 4, "row counts", (void**)&rcnt), "row counts");
  const uint32_t rblocks = (uint32_t)(((uint64_t)N * 64 + 255) / 256);
  hipLaunchKernelGGL(tg::k_rows<false>, dim3(rblocks), dim3(256), 0, st, iv, req_ptr, N, shift, bptr, bent, rcnt,
                     (const uint64_t*)nullptr, (uint32_t*)nullptr);
  ICHK(hipGetLastError(), "k_rows (count)");
  ICHK(tg::scan_counts(rcnt, N, row, ws, st), "row scan");
  ICHK(read_back(E, row + N, 8, st), "edge count read-back");
  const tg_status s = edge_buffer(ws, *E, col, alloc_col, col_cap);
  if (s != TG_OK) return s;
  if (*E) {
    hipLaunchKernelGGL(tg::k_rows<true>, dim3(rblocks), dim3(256), 0, st, iv, req_ptr, N, shift, bptr, bent, rcnt, row,
                       *col);
    ICHK(hipGetLastError(), "k_rows (fill)");
    hipLaunchKernelGGL(tg::k_sort_rows, dim3(N), dim3(256), 0, st, row, N, *col);
    ICHK(hipGetLastError(), "k_sort_rows");
  }
  ICHK(hipStreamSynchronize(st), "inference");
  return TG_OK;
}

// infer_steps with what it shares given back safely: on an error kernels may
// still be queued that store into the pinned words, or into a scratch array the
// caller is about to release, so the stream is waited for first.
tg_status infer_core(Workspace& ws, uint32_t N, uint64_t M, uint64_t space, const tg_region_req* rq,
                     const uint64_t* req_ptr, uint64_t max_buckets, hipStream_t st, uint64_t* row, uint32_t** col,
                     bool alloc_col, uint64_t col_cap, uint64_t* E) {
  const PinBlock pb(ws.spill);  // a workspace that may not allocate: no block made either
  const tg_status s = infer_steps(ws, N, M, space, rq, req_ptr, max_buckets, st, pb.p, row, col, alloc_col, col_cap, E);
  if (s != TG_OK) (void)hipStreamSynchronize(st);
  return s;
}

#undef ICHK

}  // namespace

// Finalize path: requirements from host memory, DAG back to host memory;
// device buffers allocated for the call.  One finalize infers at a time.
tg_status tg_infer_dag_host(uint32_t N, const uint64_t* req_ptr, const void* reqs, uint64_t M, uint64_t space,
                            InferResult& res) {
  res.row_ptr.assign((size_t)N + 1, 0);
  res.col.clear();
  res.ms = 0;
  if (N == 0) return TG_OK;
  static std::mutex mu;
  std::lock_guard<std::mutex> lk(mu);
  hipStream_t st = nullptr;
  hipError_t e = hipStreamCreateWithFlags(&st, hipStreamNonBlocking);
  if (e != hipSuccess) return tg_set_error(TG_EDEVICE, "hipStreamCreateWithFlags: %s", hipGetErrorString(e));
  hipEvent_t e0 = nullptr, e1 = nullptr;
  tg_status s = TG_OK;
  {
    Workspace ws;
    const SpareUse spare_use(ws, st);
    tg_region_req* d_rq = nullptr;
    uint64_t *d_req = nullptr, *d_row = nullptr;
    uint32_t* d_col = nullptr;
    uint64_t E = 0;
    if ((e = hipEventCreate(&e0)) != hipSuccess || (e = hipEventCreate(&e1)) != hipSuccess ||
        (e = ws.get(M * sizeof(tg_region_req), "requirements", (void**)&d_rq)) != hipSuccess ||
        (e = ws.get(((size_t)N + 1) * 8, "row pointers", (void**)&d_req)) != hipSuccess ||
        (e = ws.get(((size_t)N + 1) * 8, "rows", (void**)&d_row)) != hipSuccess ||
        (M && (e = hipMemcpyAsync(d_rq, reqs, M * sizeof(tg_region_req), hipMemcpyHostToDevice, st)) != hipSuccess) ||
        (e = hipMemcpyAsync(d_req, req_ptr, ((size_t)N + 1) * 8, hipMemcpyHostToDevice, st)) != hipSuccess ||
        (e = hipEventRecord(e0, st)) != hipSuccess) {
      s = tg_set_error(TG_EDEVICE, "dependence inference set-up: %s", hipGetErrorString(e));
    } else {
      s = infer_core(ws, N, M, space, d_rq, d_req, 1ull << 26, st, d_row, &d_col, true, 0, &E);
    }
    if (s == TG_OK) {
      res.col.resize(E);
      if ((e = hipEventRecord(e1, st)) != hipSuccess ||
          (e = hipMemcpyAsync(res.row_ptr.data(), d_row, ((size_t)N + 1) * 8, hipMemcpyDeviceToHost, st)) != hipSuccess ||
          (E && (e = hipMemcpyAsync(res.col.data(), d_col, E * 4, hipMemcpyDeviceToHost, st)) != hipSuccess) ||
          (e = hipStreamSynchronize(st)) != hipSuccess) {
        s = tg_set_error(TG_EDEVICE, "dependence inference read-back: %s", hipGetErrorString(e));
      } else {
        float ms = 0;
        if (hipEventElapsedTime(&ms, e0, e1) == hipSuccess) res.ms = ms;
      }
    }
    (void)hipStreamSynchronize(st);  // before the workspace's memory is given back
  }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipStreamDestroy(st);
  return s;
}

// ------------------------------------------- inference on device arrays

namespace {

tg_status infer_args(uint32_t N, const uint64_t* req_ptr, const tg_region_req* reqs, uint64_t M, uint64_t* row_ptr,
                     uint32_t* col, uint64_t col_cap, uint64_t* E) {
  if (!E) return tg_set_error(TG_EINVAL, "num_edges is NULL");
  *E = 0;
  if (!req_ptr || !row_ptr) return tg_set_error(TG_EINVAL, "req_ptr and row_ptr must be device arrays of ntasks + 1 words");
  if (M && !reqs) return tg_set_error(TG_EINVAL, "reqs is NULL but nreqs is %llu", (unsigned long long)M);
  if (col_cap && !col) return tg_set_error(TG_EINVAL, "col is NULL but col_cap is %llu", (unsigned long long)col_cap);
  // one workgroup per row sorts the rows: the grid limit bounds the task count
  if (N > 0x7FFFFFFFu) return tg_set_error(TG_EINVAL, "ntasks %u exceeds 2^31 - 1", N);
  return TG_OK;
}

// ntasks = 0: the DAG is one row pointer, 0.
tg_status infer_empty(uint64_t* row_ptr, hipStream_t st) {
  hipError_t e = tg::fill_u32((uint32_t*)row_ptr, 2, 0, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return tg_set_error(TG_EDEVICE, "dependence inference: %s", hipGetErrorString(e));
  return TG_OK;
}

}  // namespace

tg_status tg_infer_dag(uint32_t ntasks, const uint64_t* req_ptr, const tg_region_req* reqs, uint64_t nreqs,
                       uint64_t index_space, uint64_t* row_ptr, uint32_t* col, uint64_t col_cap, uint64_t* num_edges,
                       void* stream) {
  tg_status s = infer_args(ntasks, req_ptr, reqs, nreqs, row_ptr, col, col_cap, num_edges);
  if (s != TG_OK) return s;
  const hipStream_t st = (hipStream_t)stream;
  if (ntasks == 0) return infer_empty(row_ptr, st);
  Workspace ws;
  const SpareUse spare_use(ws, st);
  uint32_t* c = col;
  return infer_core(ws, ntasks, nreqs, index_space, reqs, req_ptr, 1ull << 26, st, row_ptr, &c, false,
                    col_cap, num_edges);
}

// ------------------------------------------- allocation-free inference
//
// tg_infer_dag_noalloc takes every temporary of infer_core from the scratch
// array, so the call makes no allocation.

tg_status tg_infer_dag_noalloc(uint32_t ntasks, const uint64_t* req_ptr, const tg_region_req* reqs, uint64_t nreqs,
                               uint64_t index_space, uint64_t* row_ptr, uint32_t* col, uint64_t col_cap,
                               uint64_t* num_edges, void* stream) {
  tg_status s = infer_args(ntasks, req_ptr, reqs, nreqs, row_ptr, col, col_cap, num_edges);
  if (s != TG_OK) return s;
  // the interval table, the summary and the row counts must fit before any
  // device work starts; later arrays are checked as they are carved
  const uint64_t need = round256(nreqs * sizeof(IvDev)) + 256 + round256((uint64_t)ntasks * 4);
  if (nreqs > kScratchBytes || need > kScratchBytes)
    return tg_set_error(TG_ENOMEM,
                        "allocation-free inference: %u tasks with %llu requirements need more than the %zu-byte "
                        "scratch array (at least %llu bytes)",
                        ntasks, (unsigned long long)nreqs, kScratchBytes, (unsigned long long)need);
  ScratchDev* sdp = nullptr;
  if ((s = scratch_of_device(&sdp)) != TG_OK) return s;
  ScratchDev& sd = *sdp;
  std::lock_guard<std::mutex> lk(sd.mu);
  const hipStream_t st = (hipStream_t)stream;
  if (ntasks == 0) return infer_empty(row_ptr, st);
  Workspace ws;
  ws.spill = false;
  ws.base = (uint8_t*)sd.ptr;
  ws.cap = kScratchBytes;
  uint32_t* c = col;
  return infer_core(ws, ntasks, nreqs, index_space, reqs, req_ptr, kNoallocMaxBuckets, st, row_ptr, &c, false,
                    col_cap, num_edges);
}
