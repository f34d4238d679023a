// Persistent task-DAG executor for gfx950 (MI355X).
//
// Algorithm 1 of the paper compiles a fixed graph into per-resource worker
// actors: each vertex keeps an atomic counter of pending in-edges, a finished
// vertex sends one COMPLETED_EDGE per out-edge (an atomic decrement), and a
// vertex runs once its counter reaches zero.  Here a worker is a wavefront
// (mapping 1) or a workgroup (mapping 2) of one persistent launch.
//
//  * Event subsystem: one u32 counter per task in HBM, reset from the
//    in-degree before each execution and decremented once per edge with a
//    device-scope atomic.  A task is ready exactly when its counter is 0.
//  * Ready subsystem: the compiler hands every worker its own list of
//    positions in dependence-level order.  A worker polls the counters of
//    the next `window` (<= 64) unfinished positions of its list with one
//    lane per position, compacts the ready ones with a wave ballot, runs them
//    in list order and slides the window past the finished prefix.  No
//    address is shared between workers except the counters of real edges,
//    so there is no contended queue head or tail (a single-address device
//    atomic costs about 11 ns on this part; distinct addresses sustain
//    about 27 G atomics/s).
//    Polling, taking and signalling run in scalar registers, and every
//    memory round trip of a task has other work behind it (k_exec_wave).  A
//    stencil of 1024 x 500 tasks with 256-word payloads and no mix rounds
//    takes 1.9 us a level; with vector-register state, returning edge atomics
//    and the digest before the signals it took 2.75 us.
//  * Publication: payload and array writes use device-coherent (sc1)
//    stores; before the first out-edge decrement the worker waits for all
//    its stores to complete (s_waitcnt vmcnt(0)).  Readers load with sc1.
//    This avoids the L2 write-back that an agent-scope release fence issues
//    on gfx950, which costs about 13 ns per publication device-wide.
//  * Every wait is bounded: a worker whose wait has lasted the watchdog
//    interval aborts the launch only if no worker anywhere has started a
//    task for that long (workers publish a device-wide progress stamp, at
//    most once per 1/16 of the interval each); every other worker returns
//    when it sees the abort flag.  A long critical path that keeps most
//    workers idle therefore never trips the watchdog while it advances.
#include "tg_internal.h"
#include "tg_mix.h"

namespace tg {

constexpr int kSC1 = 16;  // buffer cache policy: device-scope coherent access

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t nbytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, nbytes, 0x00020000);
}

// Wait until every outstanding vector memory operation of this wave has
// completed; the memory clobber keeps the compiler from moving memory
// operations across it.  The builtin says the same (vmcnt 0, the other
// counters unlimited) to the pass that inserts waits, which does not look
// into the asm: loads issued before the drain need no wait after it.
__device__ __forceinline__ void vm_drain() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);
  asm volatile("" ::: "memory");
}

// Read-only tables (records, graph table, predecessor addresses, requirement
// lists) are read through the constant address space so that wave-uniform
// accesses become scalar loads.
// (The host compilation pass sees plain pointers.)
#if defined(__HIP_DEVICE_COMPILE__)
template <class T>
using cptr = const T __attribute__((address_space(4)))*;
#else
template <class T>
using cptr = const T*;
#endif
template <class T>
__device__ __forceinline__ cptr<T> as_const(const T* p) {
  return (cptr<T>)p;
}
__device__ __forceinline__ uint32_t uni(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ uint32_t ld_coherent(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_coherent(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------- hashing

__device__ __forceinline__ uint64_t sm64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
// low 32 bits of sm64(key ^ idx), key = sm64(seed ^ (stream << 32))
__device__ __forceinline__ uint32_t h32k(uint64_t key, uint64_t idx) { return (uint32_t)sm64(key ^ idx); }

// Wrap-around sum over the 64 lanes (all active), returned wave-uniform.
// Cross-lane moves within each 16-lane row use DPP (swap neighbours, swap
// pairs, mirror each half-row, mirror the row); the four row sums are then
// read with readlane.  No LDS round trip: this sits between a task's payload
// store and its digest store, on the task's critical path.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
  v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
  v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, false);  // row_half_mirror
  v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, false);  // row_mirror
  return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) +
         __builtin_amdgcn_readlane(v, 48);
}

// ------------------------------------------------------------------ teams

// A team is the set of lanes that executes one task: one wavefront, one
// workgroup, or (gang) the same lane slot of several workgroups on different
// CUs.  t / size() index the lanes of this wavefront or workgroup: sum()
// returns the wrap-around sum of v over them to every lane and sync() is
// their barrier.  wt() / ws() index the task's work items over the whole
// team (equal to t / size() except in a gang).
struct WaveTeam {
  uint32_t t;
  static constexpr uint32_t S = 64;
  __device__ __forceinline__ uint32_t size() const { return 64; }
  __device__ __forceinline__ uint32_t wt() const { return t; }
  __device__ __forceinline__ uint32_t ws() const { return 64; }
  __device__ __forceinline__ uint32_t sum(uint32_t v) const { return wave_sum(v); }
  __device__ __forceinline__ uint32_t digest_sum(uint32_t v) const { return wave_sum(v); }
  __device__ __forceinline__ void sync() const {}
  __device__ __forceinline__ bool leader() const { return t == 0; }
};

struct BlockTeam {
  uint32_t t, n;
  uint32_t* lds;  // 32 words: partial sums of sum() and, from 16, of the digest
  __device__ __forceinline__ uint32_t size() const { return n; }
  __device__ __forceinline__ uint32_t wt() const { return t; }
  __device__ __forceinline__ uint32_t ws() const { return n; }
  __device__ __forceinline__ void sync() const { __syncthreads(); }
  __device__ __forceinline__ bool leader() const { return t == 0; }
  // At most once a task: the barrier before the edge signals (complete_edges)
  // stands between the reads of one task's sum and the writes of the next one's.
  __device__ uint32_t sum(uint32_t v) const {
    put_sum(v, 0);
    __syncthreads();
    return get_sum(0);
  }
  __device__ uint32_t digest_sum(uint32_t v) const {
    put_sum(v, 16);
    __syncthreads();
    return get_sum(16);
  }
  __device__ __forceinline__ void put_sum(uint32_t v, uint32_t at) const {
    v = wave_sum(v);
    if ((t & 63) == 0) lds[at + (t >> 6)] = v;
  }
  __device__ __forceinline__ uint32_t get_sum(uint32_t at) const {
    const uint32_t i = t & 63u;
    return wave_sum(i < (n >> 6) ? lds[at + i] : 0u);
  }
};

// One workgroup (member m of G) of a gang: reductions and barriers stay
// inside the workgroup, work items are split over all G workgroups.
struct GangTeam : BlockTeam {
  uint32_t m, G;
  __device__ __forceinline__ uint32_t wt() const { return m * n + t; }
  __device__ __forceinline__ uint32_t ws() const { return G * n; }
  __device__ __forceinline__ bool leader() const { return m == 0 && t == 0; }
};

// ----------------------------------------------------------------- record

__device__ __forceinline__ uint32_t rl(uint32_t v, uint32_t k) { return __builtin_amdgcn_readlane(v, k); }

// A task record as one team holds it: every wavefront loads the 128-byte
// record with one coalesced load (lane i: dword i % 32) and reads the scalar
// fields out with readlane.  succ0 is the successor this team index signals
// first (index t): the record's first dwords, so lanes 0-7 hold theirs already,
// and no load stands between the payload store and the edge signals.
struct Rec {
  uint32_t v;
  uint64_t out;
  uint32_t tid, graph, npred, succ_beg, nsucc, rounds, shape;
  uint32_t succ0;
  uint32_t* digest;  // the graph's digests
};

// This lane's dword of the record at `pos`.  Records are read-only while a
// launch runs, so a plain (cached) load is enough.
__device__ __forceinline__ uint32_t rec_dword(const ExecParams& P, uint32_t pos, uint32_t lane) {
  return reinterpret_cast<const uint32_t*>(P.rec + pos)[lane & 31u];
}

template <class Team>
__device__ __forceinline__ void unpack_rec(const Team& tm, const ExecParams& P, uint32_t v, Rec& r) {
  r.v = v;
  r.out = (uint64_t)rl(r.v, kDwOut) | ((uint64_t)rl(r.v, kDwOut + 1) << 32);
  r.tid = rl(r.v, kDwTid);
  r.graph = rl(r.v, kDwGraph);
  r.npred = rl(r.v, kDwNpred);
  r.succ_beg = rl(r.v, kDwSuccBeg);
  r.nsucc = rl(r.v, kDwNsucc);
  r.rounds = rl(r.v, kDwRounds);
  r.shape = rl(r.v, kDwShape);
  r.digest = as_const(P.gtab)[r.graph].digest;
  r.succ0 = r.v;
  if (r.nsucc > kInSucc) {
    const uint32_t s = P.succ_pos[r.succ_beg + min(tm.t, r.nsucc - 1u)];
    if (tm.t >= kInSucc) r.succ0 = s;
  }
}

// Payload address of predecessor j (j wave-uniform).
__device__ __forceinline__ uint64_t pred_at(const ExecParams& P, const Rec& r, uint32_t j) {
  if (j < kInPred) return (uint64_t)rl(r.v, kDwPred + 2 * j) | ((uint64_t)rl(r.v, kDwPred + 2 * j + 1) << 32);
  return as_const(P.pred_addr)[rl(r.v, kDwPredBeg) + j];
}

// ------------------------------------------------------------------ bodies

template <int VEC>
struct VecT;
template <>
struct VecT<1> { typedef uint32_t T; };
template <>
struct VecT<2> { typedef u32x2 T; };
template <>
struct VecT<4> { typedef u32x4 T; };

template <int VEC>
__device__ __forceinline__ typename VecT<VEC>::T buf_load(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  if constexpr (VEC == 4) return __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, 0, kSC1);
  else if constexpr (VEC == 2) return __builtin_amdgcn_raw_buffer_load_b64(r, byte_off, 0, kSC1);
  else return __builtin_amdgcn_raw_buffer_load_b32(r, byte_off, 0, kSC1);
}
template <int VEC>
__device__ __forceinline__ void buf_store(typename VecT<VEC>::T v, __amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  if constexpr (VEC == 4) __builtin_amdgcn_raw_buffer_store_b128(v, r, byte_off, 0, kSC1);
  else if constexpr (VEC == 2) __builtin_amdgcn_raw_buffer_store_b64(v, r, byte_off, 0, kSC1);
  else __builtin_amdgcn_raw_buffer_store_b32(v, r, byte_off, 0, kSC1);
}

template <int VEC>
__device__ __forceinline__ uint32_t elem(typename VecT<VEC>::T v, int i) {
  if constexpr (VEC == 1) return v;
  else return v[i];
}

// Called by a body once its first loads are issued: the list executors fetch
// the record of the next task there, behind loads the body waits for anyway.
struct NoPrefetch {
  __device__ __forceinline__ void operator()() const {}
};

// The input of one chunk (words k0 .. k0 + VEC - 1 of every lane) of a task of
// at most five predecessors: all loads issued together, one memory round trip.
template <int VEC, class Prefetch>
__device__ __forceinline__ typename VecT<VEC>::T gather5(const ExecParams& P, const Rec& r, uint32_t nbytes,
                                                         uint32_t k0, Prefetch&& prefetch) {
  typedef typename VecT<VEC>::T V;
  auto in = [&](uint32_t j) { return buf_load<VEC>(make_rsrc((const void*)pred_at(P, r, j), nbytes), k0 * 4u); };
  const V p0 = in(0);
  if (r.npred == 1) {
    prefetch();
    return p0;
  }
  const V p1 = in(1);
  if (r.npred == 2) {
    prefetch();
    return p0 + p1;
  }
  const V p2 = in(2);
  if (r.npred == 3) {
    prefetch();
    return p0 + p1 + p2;
  }
  const V p3 = in(3);
  if (r.npred == 4) {
    prefetch();
    return (p0 + p1) + (p2 + p3);
  }
  const V p4 = in(4);
  prefetch();
  return ((p0 + p1) + (p2 + p3)) + p4;
}

// Issue priority of a wavefront (0, the lowest, is the default).  A SIMD's
// wavefronts share its issue slots by priority, not evenly.  At 3: the scheduling,
// payload and signal phases, and mixes of fewer than 32 rounds, which are a few
// instructions between memory round trips and which other tasks wait for.  Mixes
// of 32 rounds or more by their length, long ones first, since a chain of them is
// what a launch of uneven graphs ends with: 2, 1, and 0 for the short ones, which
// then share with the polls of waiting workers (0 too, but mostly asleep).
// 48 graphs of log-normal costs over 4096
// workers: 31.9 ms, with equal priorities 38.4 (with all three mix classes at one
// priority 35.3, with polls at the highest 34.2); the 1024-column halo program on
// gangs 16.1 ms, 16.7 with equal ones.  The thresholds are rounds times words per lane:
// about 5 us and 80 us of a SIMD's time.
// Kernels of other streams on the same SIMD are at 0.  Beside 4096 workers (half of
// them all) with tasks of 1024 rounds a function in 64-bit floats takes 12.4 times its
// time alone, a matrix product 8.7 and an addition 2.8 times; beside the same
// executor without priorities 11.0, 7.8 and 2.6 times; with 31 rounds or 2048 workers
// there is no difference.  It is the mixes at 1 and 2 that cost this: with all of
// them at 0 it is gone, and the 48 graphs' call takes 39.7 ms instead of 33.0.
constexpr uint32_t kPrioPoll = 0, kPrioShort = 3;

// Around the mix of a task of `len` words on S lanes (of one chunk, or of all: once
// a chunk cost a 64 KiB stencil 3% of its time and halo tasks 1%).
struct MixPriority {
  uint32_t R, S;
  uint64_t len;
  __device__ __forceinline__ void operator()(bool begin) const {
    if (!begin) {
      __builtin_amdgcn_s_setprio(kPrioShort);
    } else if (R >= 32u) {
      const uint32_t w = min(R, 4095u) * (uint32_t)min(len, (uint64_t)0xFFFFFu);
      if (w < S << 9) __builtin_amdgcn_s_setprio(0);
      else if (w < S << 13) __builtin_amdgcn_s_setprio(1);
      else __builtin_amdgcn_s_setprio(2);
    }
  }
};

// A task of NP predecessors whose payload takes several chunks, two chunks at
// a time: the loads of both are in flight together, so a payload costs one
// memory round trip per two chunks.  Up to three predecessors, whose two chunks
// take 24 vector registers; four or five would spill.  192 x 40 stencil tasks of
// 64 KiB (about 0.2 ms of traffic) took 415 us on four wavefronts each, 749 us
// one chunk at a time, and 512 x 200 of 4 KiB on one wavefront 543 and 975 us
// (432 and 543 us since the mix is unrolled and the barriers are two).
// Issuing the next pair's loads before this pair's mix as well spills too: 367
// us for the former, 635 us for the latter.
template <int VEC, int NP, class Team, class Prefetch>
__device__ __forceinline__ uint32_t explicit_chunks(const Team& tm, const ExecParams& P, const Rec& r, uint32_t n,
                                                    Prefetch&& prefetch) {
  typedef typename VecT<VEC>::T V;
  const uint32_t nbytes = n * 4u, step = VEC * tm.ws();
  const uint32_t pairs = uni((n + 2u * step - 1u) / (2u * step));
  uint32_t k0 = tm.wt() * VEC, dsum = 0;
  const MixPriority prio{r.rounds, tm.ws(), n};
  prio(true);
  for (uint32_t c = 0; c < pairs; ++c) {
    V p[NP], q[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      const __amdgpu_buffer_rsrc_t in = make_rsrc((const void*)pred_at(P, r, j), nbytes);
      p[j] = buf_load<VEC>(in, k0 * 4u);
      q[j] = buf_load<VEC>(in, (k0 + step) * 4u);
    }
    if (c == 0) prefetch();
#pragma unroll
    for (int j = 1; j < NP; ++j) {
      p[0] += p[j];
      q[0] += q[j];
    }
    const __amdgpu_buffer_rsrc_t wr = make_rsrc((const void*)r.out, nbytes);
    const V x = mix_rounds(V(p[0] ^ r.tid), r.rounds);
    buf_store<VEC>(x, wr, k0 * 4u);
    const V y = mix_rounds(V(q[0] ^ r.tid), r.rounds);
    buf_store<VEC>(y, wr, (k0 + step) * 4u);
    uint32_t dx = 0, dy = 0;
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      dx += elem<VEC>(x, i) * (2u * (k0 + i) + 1u);
      dy += elem<VEC>(y, i) * (2u * (k0 + step + i) + 1u);
    }
    dsum += (k0 < n ? dx : 0u) + (k0 + step < n ? dy : 0u);
    k0 += 2u * step;
  }
  prio(false);
  return dsum;
}

// Explicit body over words k = k0, k0 + VEC*S, ... handled VEC at a time.
// The chunk loop and the mix-round loop have wave-uniform trip counts (n,
// the team size and R are uniform), so both run under scalar loop control.
// The buffer descriptors bound every access to the payload: a lane whose
// chunk lies past it (a team wider than n / VEC) loads zeros and stores
// nothing, and leaves the digest alone.
template <int VEC, class Team, class Prefetch>
__device__ __forceinline__ uint32_t explicit_words(const Team& tm, const ExecParams& P, const Rec& r, uint32_t n,
                                                   Prefetch&& prefetch) {
  typedef typename VecT<VEC>::T V;
  const uint32_t S = tm.ws();
  const uint32_t nbytes = n * 4u;
  const uint32_t npred = r.npred, R = r.rounds, tid = r.tid;
  const __amdgpu_buffer_rsrc_t wr = make_rsrc((const void*)r.out, nbytes);
  const uint32_t step = VEC * S;
  uint32_t dsum = 0;
  if (n <= step && npred - 1u < 5u) {
    const uint32_t k0 = tm.wt() * VEC;
    const V x = mix_rounds(V(gather5<VEC>(P, r, nbytes, k0, prefetch) ^ tid), R, MixPriority{R, S, n});
    buf_store<VEC>(x, wr, k0 * 4);
#pragma unroll
    for (int i = 0; i < VEC; ++i) dsum += elem<VEC>(x, i) * (2u * (k0 + i) + 1u);
    return k0 < n ? dsum : 0u;
  }
  if constexpr (VEC == 4)  // (narrower vectors: at most one chunk and a half)
    if (npred - 1u < 3u) {
      if (npred == 1) return explicit_chunks<VEC, 1>(tm, P, r, n, prefetch);
      if (npred == 2) return explicit_chunks<VEC, 2>(tm, P, r, n, prefetch);
      return explicit_chunks<VEC, 3>(tm, P, r, n, prefetch);
    }
  const uint32_t chunks = uni((n + step - 1u) / step);
  for (uint32_t c = 0; c < chunks; ++c) {
    const uint32_t k0 = c * step + tm.wt() * VEC;
    V acc = V(0);
    if (npred == 0) {
      if (c == 0) prefetch();
      // source: initial payload from the graph seed
      const uint64_t key = as_const(P.gtab)[r.graph].key1;
      if constexpr (VEC == 1) {
        acc = h32k(key, ((uint64_t)tid << 16) | k0);
      } else {
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = h32k(key, ((uint64_t)tid << 16) | (k0 + i));
      }
    } else {
      // groups of up to five predecessors, each group's loads issued
      // together: one memory round trip per group, not per predecessor
      uint32_t j = 0;
      while (j < npred) {
        const uint32_t m = npred - j;  // wave-uniform
        const bool first = (c | j) == 0u;
        auto in = [&](uint32_t i) {
          return buf_load<VEC>(make_rsrc((const void*)pred_at(P, r, j + i), nbytes), k0 * 4);
        };
        if (m >= 5) {
          const V p0 = in(0), p1 = in(1), p2 = in(2), p3 = in(3), p4 = in(4);
          if (first) prefetch();
          acc += ((p0 + p1) + (p2 + p3)) + p4;
          j += 5;
        } else if (m == 4) {
          const V p0 = in(0), p1 = in(1), p2 = in(2), p3 = in(3);
          if (first) prefetch();
          acc += (p0 + p1) + (p2 + p3);
          j += 4;
        } else if (m == 3) {
          const V p0 = in(0), p1 = in(1), p2 = in(2);
          if (first) prefetch();
          acc += (p0 + p1) + p2;
          j += 3;
        } else if (m == 2) {
          const V p0 = in(0), p1 = in(1);
          if (first) prefetch();
          acc += p0 + p1;
          j += 2;
        } else {
          const V p0 = in(0);
          if (first) prefetch();
          acc += p0;
          j += 1;
        }
      }
    }
    const V x = mix_rounds(V(acc ^ tid), R, MixPriority{R, S, n});
    buf_store<VEC>(x, wr, k0 * 4);
    if (k0 < n) {
#pragma unroll
      for (int i = 0; i < VEC; ++i) dsum += elem<VEC>(x, i) * (2u * (k0 + i) + 1u);
    }
  }
  return dsum;
}

// Returns this lane's digest part.
template <class Team, class Prefetch>
__device__ __forceinline__ uint32_t body_explicit(const Team& tm, const ExecParams& P, const Rec& r, uint32_t n,
                                                  Prefetch&& prefetch) {
  const uint32_t S = tm.ws();
  if (n >= 4 * S) return explicit_words<4>(tm, P, r, n, prefetch);
  if (n >= 2 * S) return explicit_words<2>(tm, P, r, n, prefetch);
  return explicit_words<1>(tm, P, r, n, prefetch);
}

// Elements t, t + S, t + 2S, t + 3S of p[0, len) (0 past the end).
__device__ __forceinline__ u32x4 load4(const uint32_t* p, uint32_t t, uint32_t S, uint64_t len) {
  u32x4 x;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint64_t o = t + (uint64_t)k * S;
    x[k] = o < len ? ld_coherent(p + o) : 0u;
  }
  return x;
}

// Returns this lane's digest part.  Every workgroup of a gang sums all
// read-only elements itself; the read-write elements are split over the gang.
template <class Team, class Prefetch>
__device__ __forceinline__ uint32_t body_implicit(const Team& tm, const ExecParams& P, const Rec& r,
                                                  Prefetch&& prefetch) {
  const cptr<ReqDev> rq = as_const((const ReqDev*)r.out);
  const uint32_t nreq = rl(r.v, kDwNreq);
  uint32_t* const A = as_const(P.gtab)[r.graph].data;
  // read-only elements: their wrap sum c
  uint32_t part = 0;
  for (uint32_t i = 0; i < nreq; ++i) {
    const ReqDev q = rq[i];
    if (q.priv != 1) continue;
    for (uint64_t e = q.lo + tm.t; e < q.hi; e += tm.size()) part += ld_coherent(A + e);
  }
  prefetch();
  const uint32_t key = uni(tm.sum(part) ^ r.tid);
  const uint32_t R = r.rounds;
  const uint32_t S = tm.ws(), wt = tm.wt();
  uint32_t dsum = 0;
  for (uint32_t i = 0; i < nreq; ++i) {
    const ReqDev q = rq[i];
    if (q.priv != 2) continue;
    const uint64_t len = q.hi - q.lo;
    uint32_t* const a = A + q.lo;
    // four elements per lane per chunk; the chunk loop and the mix-round
    // loop are wave-uniform, lanes past the end skip loads and stores; the
    // next chunk's loads are issued before this chunk's mix
    const uint64_t step = 4 * (uint64_t)S;
    u32x4 x = load4(a, wt, S, len);
    const MixPriority prio{R, S, len};
    prio(true);
    for (uint64_t base = 0; base < len; base += step) {
      const u32x4 y = base + step < len ? load4(a + base + step, wt, S, len - base - step) : u32x4{0, 0, 0, 0};
      x = mix_rounds(u32x4(x ^ key), R);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint64_t o = base + wt + (uint64_t)k * S;
        if (o < len) {
          st_coherent(a + o, x[k]);
          dsum += x[k] * (2u * (q.rw_base + (uint32_t)o) + 1u);
        }
      }
      x = y;
    }
    prio(false);
  }
  return dsum;
}

// Run the task at `pos`, whose unpacked record is r.  Returns this lane's
// digest part.  DIAG: a diagnostic launch (start times, run counts).
template <bool DIAG, class Team, class Prefetch>
__device__ __forceinline__ uint32_t run_body(const Team& tm, const ExecParams& P, uint32_t pos, const Rec& r,
                                             Prefetch&& prefetch) {
  if (DIAG && P.tstamp && tm.leader()) P.tstamp[2 * pos] = __builtin_amdgcn_s_memrealtime();
  const uint32_t d = (r.shape >> 24) == 1u ? body_explicit(tm, P, r, r.shape & 0xFFFFFFu, prefetch)
                                           : body_implicit(tm, P, r, prefetch);
  if (DIAG && P.execs && tm.leader())
    __hip_atomic_fetch_add(P.execs + pos, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return d;
}

// Stores a task's digest: the sum of its lanes' parts.  Device-coherent, so it
// is in memory once the leader's stores are drained.
template <class Team>
__device__ __forceinline__ void store_digest(const Team& tm, const Rec& r, uint32_t part) {
  const uint32_t d = tm.digest_sum(part);
  if (tm.leader()) st_coherent(r.digest + r.tid, d);
}

// Signal one out-edge of a finished task (COMPLETED_EDGE).  Nothing waits for
// the decrement unless doorbells are on (NOTIFY): then, for the edge that
// empties a counter, the message that starts the task at its owner follows --
// the owner's doorbell is rung only after the decrement has been performed (its
// old value has returned).  The two forms are separate kernels: as a branch on
// a parameter the compiler merged them into one returning atomic, and every
// task waited for it (about 1100 cycles).
template <bool NOTIFY>
__device__ __forceinline__ void signal_edge(const ExecParams& P, uint32_t dst) {
  if (NOTIFY && P.notify) {
    const uint32_t old = __hip_atomic_fetch_sub(P.cnt + dst, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((old & kPendingMask) == 1u)
      __hip_atomic_fetch_add(P.bell + P.owner[dst] * kBellStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    (void)__hip_atomic_fetch_sub(P.cnt + dst, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

template <bool NOTIFY, class Team>
__device__ __forceinline__ void complete_edges(const Team& tm, const ExecParams& P, const Rec& r) {
  vm_drain();  // this lane's payload stores are complete
  tm.sync();   // ... and so are every other lane's of the team
  if (tm.t < r.nsucc) signal_edge<NOTIFY>(P, r.succ0);
  if (r.nsucc > tm.size())
    for (uint32_t j = tm.t + tm.size(); j < r.nsucc; j += tm.size())
      signal_edge<NOTIFY>(P, P.succ_pos[r.succ_beg + j]);
}

// A launch behind a pre-condition wait (k_wait_flags) does nothing if the
// wait gave up: the wait raised the abort flag, which the reset before it
// had cleared.
__device__ __forceinline__ bool gate_closed(const ExecParams& P) {
  return P.gated && uni(ld_coherent(&P.ctrl->abort)) != 0u;
}

// ------------------------------------------------------------ worker loop

constexpr uint32_t kExit = 0xFFFFFFFFu;

// Per-worker scheduling state, the same in all lanes of the wave that runs the
// state machine, and kept in scalar registers: no branch of it may depend on a
// lane in a way that leaves its loops (a lane-dependent report before a return
// once did, and the compiler then kept all of this in vector registers under
// execution masks: about 1700 cycles a task).
struct WorkerState {
  uint32_t worker, wb, wcnt;  // list of positions [wb, wb + wcnt)
  uint32_t h;                 // first unfinished list entry
  uint64_t done;              // bit i: entry h + i already taken
  uint64_t pend;              // ready entries found by the last scan, not yet taken
  uint32_t seen;              // last doorbell value read
  uint32_t spins;             // consecutive empty polls
  uint64_t now;               // clock at the last scan, or at the last task taken after it
  bool fresh;                 // `now` is of this scan: no task taken since
  uint64_t last;              // time of the last task taken (realtime counter)
  uint64_t pub;               // time this worker last published Ctrl::progress
  uint32_t stop;              // why next_task returned kExit (kGoOn: the list is finished)
  uint32_t pf_pos;            // position whose record dword is held in pf_v
  uint32_t pf_v;              // per lane: dword lane % 32 of that record
};
// Results of an empty poll.
constexpr uint32_t kGoOn = 0, kLeave = 1, kStuck = 2;

__device__ __forceinline__ uint64_t uni64(uint64_t x) {
  return ((uint64_t)uni((uint32_t)(x >> 32)) << 32) | uni((uint32_t)x);
}

// Fetches the record of the entry likeliest to run next: the first one found
// ready and not yet taken, else the oldest one not taken (past the end of the
// list, the last one again: the load is unconditional, so that the compiler
// counts exactly how many younger loads an earlier one need not wait for).
__device__ __forceinline__ void fetch_next(const ExecParams& P, WorkerState& w, uint32_t lane) {
  const uint64_t u = w.pend ? w.pend : ~w.done;
  const uint32_t e = w.h + (u ? (uint32_t)__builtin_ctzll(u) : 64u);
  w.pf_pos = w.wb + min(e, w.wcnt - 1u);
  w.pf_v = rec_dword(P, w.pf_pos, lane);
}

// One poll of the ready window: every lane reads one counter and ballots
// collect the ready entries.  Lanes past the window read
// its last counter again.  SCANREC: also fetch the record of the oldest
// unfinished entry in the same round trip (once per entry); the wavefront
// executor has fetched it during the task before.
// What is left to do while the counters are on their way: `overlap`.
template <bool SCANREC, class Overlap>
__device__ __forceinline__ uint64_t ready_scan(uint32_t lane, const ExecParams& P, WorkerState& w,
                                               Overlap&& overlap) {
  const uint32_t n = min(w.wcnt - w.h, P.window);
  const uint32_t c = ld_coherent(P.cnt + w.wb + w.h + min(lane, n - 1u));
  if (SCANREC) {
    const uint32_t head = w.wb + w.h;
    if (head != w.pf_pos) {
      w.pf_v = rec_dword(P, head, lane);
      w.pf_pos = head;
    }
  }
  w.now = __builtin_amdgcn_s_memrealtime();
  w.fresh = true;
  overlap();
  const uint64_t zero = __ballot((c & kPendingMask) == 0u) & ~w.done & (n < 64u ? (1ull << n) - 1ull : ~0ull);
  // an entry marked kAfterPrev also needs the entry before it taken (entry
  // h - 1 is finished; this worker runs its tasks one after another)
  return uni64(zero & (~__ballot((int)c < 0) | w.done << 1 | 1ull));
}

// Global progress: a worker that takes a task publishes the time (atomic
// max on one word), at most once per progress_ticks, so the word is written
// rarely however many tasks run.
__device__ __forceinline__ void publish_progress(const ExecParams& P, WorkerState& w, uint32_t lane) {
  if (w.now - w.pub < P.progress_ticks) return;
  w.pub = w.now;
  if (lane == 0) __hip_atomic_fetch_max(&P.ctrl->progress, w.now, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// True when nothing has progressed for the watchdog interval: neither this
// wait (which began at `since`) nor any worker's published task start is
// more recent than watchdog_ticks before `now`.  Clocks read by different
// waves may differ slightly, so a stamp later than `now` counts as `now`.
__device__ __forceinline__ bool stalled(const ExecParams& P, uint64_t since, uint64_t now) {
  if (now - since <= P.watchdog_ticks) return false;
  uint64_t g = __hip_atomic_load(&P.ctrl->progress, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  g = ((uint64_t)uni((uint32_t)(g >> 32)) << 32) | uni((uint32_t)g);
  if (g > now) return false;
  return now - g > P.watchdog_ticks;
}

// Back-off after `spins` consecutive empty polls, in naps of 128 cycles (55
// ns): one nap for the first polls, then a quarter of their number up to 16,
// so that a wake-up comes late by a small part of the wait; from the 64th on
// idle_sleep naps (at least those 16), doubling after every further 64 empty
// polls up to 32 x idle_sleep (at most 256 naps, 14 us).  A worker waiting for a
// quick hand-off polls again at once; one waiting behind a long task soon polls
// only every few microseconds, and so stops taking issue slots from the waves
// on its SIMD that run tasks, and memory from everybody: an empty poll takes
// 0.2 us, and thousands of workers that kept polling at that rate slowed every
// hand-off (a 1024 x 200 stencil in level order over 8192 workers: 3.49 ms at
// one nap a poll, 0.54 ms so).
__device__ __forceinline__ void idle_nap(const ExecParams& P, uint32_t spins) {
  uint32_t nap = max(1u, min(spins >> 2, 16u));
  if (spins >= 64) nap = max(nap, min(P.idle_sleep << min((spins >> 6) - 1u, 5u), 256u));
  for (uint32_t i = 0; i < nap; ++i) __builtin_amdgcn_s_sleep(2);
}

// One empty poll: back off, and every 64 polls check the abort flag and the
// watchdog.
__device__ __forceinline__ uint32_t idle_step(const ExecParams& P, WorkerState& w) {
  ++w.spins;
  __builtin_amdgcn_s_setprio(kPrioPoll);
  idle_nap(P, w.spins);
  if ((w.spins & 63u) != 0u) return kGoOn;
  if (uni(ld_coherent(&P.ctrl->abort)) != 0u) return kLeave;
  const uint64_t now = __builtin_amdgcn_s_memrealtime();
  return stalled(P, w.last, now) || (P.spin_limit != 0u && w.spins >= P.spin_limit) ? kStuck : kGoOn;
}

// Tells the host that the abort flag has been raised: it looks at the control
// block only then.
__device__ __forceinline__ void raise_alarm(uint32_t* alarm) {
  if (alarm) __hip_atomic_store(alarm, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// A worker that found no progress raises the abort flag; the first one
// records where it was stuck.
__device__ __forceinline__ void report_stuck(const ExecParams& P, const WorkerState& w, uint32_t lane) {
  if (w.stop != kStuck || lane != 0) return;
  const uint32_t prev = __hip_atomic_fetch_add(&P.ctrl->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (prev == 0u) {
    st_coherent(&P.ctrl->stuck_worker, w.worker);
    st_coherent(&P.ctrl->stuck_pos, w.wb + w.h);
    st_coherent(&P.ctrl->stuck_cnt, ld_coherent(P.cnt + w.wb + w.h));
    st_coherent(&P.ctrl->stuck_h, w.h);
    st_coherent(&P.ctrl->stuck_wcnt, w.wcnt);
  }
  raise_alarm(P.alarm);
}

// Diagnostics of one poll: first and last time, number.
__device__ __forceinline__ void stamp_scan(const ExecParams& P, const WorkerState& w, uint32_t lane) {
  if (!P.wstamp || lane != 0) return;
  uint64_t* ws = P.wstamp + 4 * w.worker;
  const uint64_t now = __builtin_amdgcn_s_memrealtime();
  if (ws[0] == 0) ws[0] = now;
  ws[1] = now;
  ws[2] += 1;
}

// Returns the position of the worker's next ready task, or kExit when its
// list is finished or the launch is being aborted (w.stop says which).  Run by
// one whole wave.  FULL: doorbells and diagnostics may be on.  The first poll
// after a task has `overlap` to do meanwhile; the polls after it, should it find
// nothing, are a loop of their own of few instructions, since they take issue
// slots from the waves that run tasks.
template <bool FULL, bool SCANREC, class Overlap>
__device__ __forceinline__ uint32_t next_task(const ExecParams& P, WorkerState& w, uint32_t lane, Overlap&& overlap) {
  for (;;) {
    if (w.pend) {
      const uint32_t b = (uint32_t)__builtin_ctzll(w.pend);
      w.pend &= w.pend - 1;
      w.done |= 1ull << b;
      w.spins = 0;
      if (!w.fresh) {
        w.now = __builtin_amdgcn_s_memrealtime();
        overlap();
      }
      w.fresh = false;
      w.last = w.now;
      publish_progress(P, w, lane);
      return w.wb + w.h + b;
    }
    // slide the window past the finished prefix
    const uint32_t adv = (~w.done == 0ull) ? 64u : (uint32_t)__builtin_ctzll(~w.done);
    w.h += adv;
    w.done = adv >= 64u ? 0ull : (w.done >> adv);
    if (w.h >= w.wcnt) return kExit;
    w.pend = ready_scan<SCANREC>(lane, P, w, overlap);
    if (FULL) stamp_scan(P, w, lane);
    if (w.pend) continue;
    do {
      if (FULL && P.notify) {
        // wait for a message: one word per poll instead of the whole window
        // (a message rung before the last scan shows as a new value here, and
        // costs one scan)
        for (;;) {
          const uint32_t b = uni(ld_coherent(P.bell + w.worker * kBellStride));
          if (b != w.seen) {
            w.seen = b;
            break;
          }
          w.stop = idle_step(P, w);
          if (w.stop != kGoOn) return kExit;
        }
      } else {
        w.stop = idle_step(P, w);
        if (w.stop != kGoOn) return kExit;
      }
      w.pend = ready_scan<SCANREC>(lane, P, w, [] {});
      if (FULL) stamp_scan(P, w, lane);
    } while (!w.pend);
    __builtin_amdgcn_s_setprio(kPrioShort);
  }
}

// Residency probe: every worker checks in and then waits (for at most the
// watchdog interval) until all nworkers have checked in.  A worker that saw
// all of them counts itself as resident; the host accepts the worker count
// only if every worker did.  The same kernel (same resources) as the
// executor is used, so the answer holds for the real launch.
__device__ void residency_probe(const ExecParams& P, bool lead) {
  if (lead) __hip_atomic_fetch_add(&P.ctrl->started, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
  for (;;) {
    const uint32_t n = uni(ld_coherent(&P.ctrl->started));
    if (n >= P.nworkers) {
      if (lead) __hip_atomic_fetch_add(&P.ctrl->resident, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    if (__builtin_amdgcn_s_memrealtime() - t0 > P.watchdog_ticks) return;
    __builtin_amdgcn_s_sleep(8);
  }
}

__device__ __forceinline__ void worker_init(WorkerState& w, const ExecParams& P, uint32_t worker) {
  __builtin_amdgcn_s_setprio(kPrioShort);
  w.worker = worker;
  w.wb = as_const(P.wbase)[worker];
  w.wcnt = as_const(P.wbase)[worker + 1] - w.wb;
  w.h = 0;
  w.done = 0;
  w.pend = 0;
  w.seen = 0;
  w.spins = 0;
  w.now = w.last = __builtin_amdgcn_s_memrealtime();
  w.fresh = false;
  w.pub = 0;
  w.stop = kGoOn;
  w.pf_pos = kExit;
  w.pf_v = 0;
}

// One wavefront per task.  A task's chain of memory round trips is: counters
// back (and the signals of the task before acknowledged: loads return in order
// behind them), payloads back, stores drained, signals out.  Everything else
// runs while one of them is under way: the record of the next task is fetched
// behind the payload loads and unpacked behind the next poll, and the digest,
// which no other task reads, is reduced and stored there too.
template <bool FULL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_exec_wave(ExecParams P) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t worker = uni((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  if (worker >= P.nworkers || gate_closed(P)) return;
  const WaveTeam tm{lane};
  if (FULL && P.diag && lane == 0)
    __hip_atomic_fetch_add(&P.ctrl->started, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  WorkerState w;
  worker_init(w, P, worker);
  if (w.wcnt) fetch_next(P, w, lane);
  Rec r;                     // the task being run, then the next one
  uint32_t r_pos = kExit;    // position of the record in r
  uint32_t part = 0;         // digest part of the last task, until it is stored ...
  uint32_t* part_of = nullptr;  // ... here (null: stored)
  // The store is issued whether or not there is a digest (to no lane then, by
  // the descriptor's bounds), so that the compiler counts it and does not wait
  // for it where it waits for the poll before it.
  auto overlap = [&] {
    buf_store<1>(tm.sum(part), make_rsrc(part_of, part_of ? 4u : 0u), lane * 4u);
    part_of = nullptr;
    if (r_pos != w.pf_pos) {
      unpack_rec(tm, P, w.pf_v, r);
      r_pos = w.pf_pos;
    }
  };
  for (;;) {
    const uint32_t pos = next_task<FULL, false>(P, w, lane, overlap);
    if (pos == kExit) break;
    if (pos != r_pos) {
      unpack_rec(tm, P, rec_dword(P, pos, lane), r);
      r_pos = pos;
    }
    part = run_body<FULL>(tm, P, pos, r, [&] { fetch_next(P, w, lane); });
    complete_edges<FULL>(tm, P, r);
    part_of = r.digest + r.tid;
    if (FULL && P.tstamp && lane == 0) P.tstamp[2 * pos + 1] = __builtin_amdgcn_s_memrealtime();
  }
  buf_store<1>(tm.sum(part), make_rsrc(part_of, part_of ? 4u : 0u), lane * 4u);
  report_stuck(P, w, lane);
  if (FULL && P.wprog && lane == 0) P.wprog[worker] = w.h;
}

// One workgroup per task: wave 0 runs the scheduling state machine and
// stages the chosen position and its record in LDS; every wave then executes
// the same sequence of barriers for each task.
// Two barriers a task: A, behind which the task is known, and B, behind which all
// payload stores are drained (complete_edges; a task with read-only elements has
// one more in their sum, whose words no other sum uses).  The position and record are written
// before A and read before B, so the next ones need no barrier of their own; the
// digest's partial sums are written after B and added up behind the next A.
// Five barriers a task before: 64 KiB stencil 447 -> 432 us, 128 x 40 butterfly of
// 64 KiB 243 -> 237 us, 1024-column halo on gangs 15.8 -> 15.6 ms.
template <bool FULL>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_exec_block(ExecParams P) {
  __shared__ uint32_t lds[32];
  __shared__ uint32_t cmd;
  __shared__ uint32_t recl[32];
  const uint32_t worker = blockIdx.x;
  if (worker >= P.nworkers || gate_closed(P)) return;
  const BlockTeam tm{threadIdx.x, blockDim.x, lds};
  const uint32_t lane = threadIdx.x & 63u, wave = uni(threadIdx.x >> 6);
  if (FULL && P.diag && threadIdx.x == 0)
    __hip_atomic_fetch_add(&P.ctrl->started, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  WorkerState w;
  worker_init(w, P, worker);
  uint32_t part = 0;            // digest part of the last task: summed over the barrier
  uint32_t* part_of = nullptr;  // behind which the next task is known, and stored here
  for (;;) {
    if (part_of) tm.put_sum(part, 16);
    if (wave == 0) {
      const uint32_t pos = next_task<FULL, true>(P, w, lane, [] {});
      if (pos != kExit) {
        const uint32_t v = pos == w.pf_pos ? w.pf_v : rec_dword(P, pos, lane);
        if (lane < 32) recl[lane] = v;
      }
      if (lane == 0) cmd = pos;
    }
    __syncthreads();
    const uint32_t pos = uni(cmd);
    const uint32_t v = recl[lane & 31u];
    if (part_of && wave == 0) {
      const uint32_t d = tm.get_sum(16);
      if (lane == 0) st_coherent(part_of, d);
    }
    if (pos == kExit) break;
    Rec r;
    unpack_rec(tm, P, v, r);
    part = run_body<FULL>(tm, P, pos, r, NoPrefetch());
    complete_edges<FULL>(tm, P, r);
    part_of = r.digest + r.tid;
    if (FULL && P.tstamp && threadIdx.x == 0) P.tstamp[2 * pos + 1] = __builtin_amdgcn_s_memrealtime();
  }
  if (wave == 0) report_stuck(P, w, lane);
  if (FULL && P.wprog && threadIdx.x == 0) P.wprog[worker] = w.h;
}

// A gang of P.gang workgroups per task (on different CUs), without a leader:
// every member runs the scheduling loop over the gang's list itself, executes
// its share of each task's work items, adds its digest part to the task's
// digest (zeroed by the reset) and signals every out-edge after draining its
// stores.  A task's counter starts at its in-degree times the gang size, so it
// becomes ready once every member of every predecessor's gang has finished
// its share.  No member waits for another: the members of one gang may run
// different tasks of the list at the same time (each takes its ready entries
// in its own order), and none of the mailbox round trips a leader would need
// (publish the task, collect the arrivals) sits between two dependent tasks.
template <bool FULL>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_exec_gang(ExecParams P) {
  __shared__ uint32_t lds[32];
  __shared__ uint32_t cmd;
  __shared__ uint32_t recl[32];
  const uint32_t G = P.gang;
  const uint32_t gang = blockIdx.x / G, member = blockIdx.x % G;
  if (gang >= P.nworkers || gate_closed(P)) return;
  GangTeam tm;
  tm.t = threadIdx.x;
  tm.n = blockDim.x;
  tm.lds = lds;
  tm.m = member;
  tm.G = G;
  const uint32_t lane = threadIdx.x & 63u, wave = uni(threadIdx.x >> 6);
  WorkerState w;
  worker_init(w, P, gang);
  uint32_t part = 0;            // digest part of the last task: summed over the barrier
  uint32_t* part_of = nullptr;  // behind which the next task is known, and stored here
  for (;;) {
    if (part_of) tm.put_sum(part, 16);
    if (wave == 0) {
      const uint32_t pos = next_task<FULL, true>(P, w, lane, [] {});
      if (pos != kExit) {
        const uint32_t v = pos == w.pf_pos ? w.pf_v : rec_dword(P, pos, lane);
        if (lane < 32) recl[lane] = v;
      }
      if (lane == 0) cmd = pos;
    }
    __syncthreads();
    const uint32_t pos = uni(cmd);
    const uint32_t v = recl[lane & 31u];
    if (part_of && wave == 0) {
      const uint32_t d = tm.get_sum(16);
      if (lane == 0) __hip_atomic_fetch_add(part_of, d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (pos == kExit) break;
    Rec r;
    unpack_rec(tm, P, v, r);
    part = run_body<FULL>(tm, P, pos, r, NoPrefetch());
    complete_edges<FULL>(tm, P, r);
    part_of = r.digest + r.tid;
    // diagnostics: a task ends when its last member finishes
    if (FULL && P.tstamp && threadIdx.x == 0)
      __hip_atomic_fetch_max(P.tstamp + 2 * pos + 1, __builtin_amdgcn_s_memrealtime(), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
  }
  if (wave == 0) report_stuck(P, w, lane);
  if (FULL && member == 0 && P.wprog && threadIdx.x == 0) P.wprog[gang] = w.h;
}

// ------------------------------------------------------ ready-queue dispatch
//
// The second dispatch of the executor (Algorithm 1's EXECUTE_OP on the
// vertex a COMPLETED_EDGE made ready), without per-worker lists.  The
// decrement that empties a counter (old value 1) makes its task ready.  A
// worker keeps the first task its own completion made ready as its next task
// (a chain causes no queue traffic) and pushes the others into one ticket
// queue shard (shards taken in turn): one ballot of the ready lanes, one
// atomic add on the shard's tail for all of them, each lane's slot from the
// count of ready lanes below it.  A worker that needs work claims a tile of
// consecutive tickets of its own shard with one atomic add on the head --
// a claim never fails and never retries -- and waits on each claimed slot in
// turn until a pusher has written it; waiting workers poll distinct slots,
// so no address is shared by the waiters.
//
// Termination needs no per-task counter: every task precedes some sink (a
// task without out-edges), so the launch is over once every sink has run.
// Workers count the sinks they finished and add the count to one word only
// when they find their next slot empty; the addition that completes the sink
// total pushes qsent exit sentinels into every shard.  A worker claims a new
// tile only after consuming its previous one, so at most one tile per worker
// (plus one straddling the last task ticket) reaches past the task tickets
// of a shard: qsent = tile x (workers of the shard + 1) sentinels fill every
// ticket ever claimed.  No worker waits for a particular other worker, so
// this dispatch needs no co-residency.

struct QueueState {
  uint32_t worker, shard, pshard;  // claims from `shard`; next push into `pshard`
  uint32_t local;                  // ready task kept by this worker (kExit: none)
  uint32_t tile_h, tile_n, tile_i; // claimed tickets [tile_h, tile_h + tile_n), next tile_i
  uint32_t sinks;                  // sinks finished since the last report
  uint64_t pub;                    // time this worker last published Ctrl::progress
  uint32_t stop;                   // kStuck: queue_next gave up at ticket `stuck`
  uint32_t stuck;
};

__device__ __forceinline__ uint32_t* q_head(const ExecParams& P, uint32_t s) { return P.qctl + s * kQLine; }
__device__ __forceinline__ uint32_t* q_tail(const ExecParams& P, uint32_t s) {
  return P.qctl + (P.qshards + s) * kQLine;
}
__device__ __forceinline__ uint32_t* q_sinks(const ExecParams& P) { return P.qctl + 2u * P.qshards * kQLine; }

// Workgroups are dealt to the 8 XCDs round-robin by workgroup index.
__device__ __forceinline__ void queue_init(QueueState& q, const ExecParams& P, uint32_t worker) {
  __builtin_amdgcn_s_setprio(kPrioShort);
  q.worker = worker;
  q.shard = blockIdx.x & 7u & (P.qshards - 1u);
  q.pshard = q.shard;
  q.local = kExit;
  q.tile_h = q.tile_n = q.tile_i = 0;
  q.sinks = 0;
  q.pub = 0;
  q.stop = kGoOn;
  q.stuck = 0;
}

// Raises the abort flag; the first abort records where it happened.
__device__ void queue_abort(const ExecParams& P, const QueueState& q, uint32_t lane, uint32_t ticket) {
  if (lane != 0) return;
  const uint32_t prev = __hip_atomic_fetch_add(&P.ctrl->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (prev == 0u) {
    st_coherent(&P.ctrl->stuck_worker, q.worker);
    st_coherent(&P.ctrl->stuck_pos, ticket);
    st_coherent(&P.ctrl->stuck_cnt, ld_coherent(q_sinks(P)));
    st_coherent(&P.ctrl->stuck_h, q.shard);
    st_coherent(&P.ctrl->stuck_wcnt, P.npos);
  }
  raise_alarm(P.alarm);
}

// The end of the launch: qsent exit sentinels into every shard.
__device__ void queue_finish(const ExecParams& P, uint32_t lane) {
  for (uint32_t s = 0; s < P.qshards; ++s) {
    uint32_t base = 0;
    if (lane == 0) base = __hip_atomic_fetch_add(q_tail(P, s), P.qsent, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    base = rl(base, 0);
    uint32_t* slot = P.q + (size_t)s * P.qcap;
    for (uint32_t i = lane; i < P.qsent; i += 64u)
      if (base + i < P.qcap) st_coherent(slot + base + i, kQExit);
  }
}

// Reports the sinks this worker finished; the report that completes the
// total ends the launch.
__device__ __forceinline__ void queue_report(const ExecParams& P, QueueState& q, uint32_t lane) {
  if (q.sinks == 0u) return;
  uint32_t old = 0;
  if (lane == 0) old = __hip_atomic_fetch_add(q_sinks(P), q.sinks, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  old = rl(old, 0);
  const bool last = old + q.sinks == P.nsinks;
  q.sinks = 0;
  if (last) queue_finish(P, lane);
}

__device__ __forceinline__ void queue_progress(const ExecParams& P, QueueState& q, uint32_t lane) {
  const uint64_t now = __builtin_amdgcn_s_memrealtime();
  if (now - q.pub < P.progress_ticks) return;
  q.pub = now;
  if (lane == 0) __hip_atomic_fetch_max(&P.ctrl->progress, now, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Position of the worker's next task, or kExit at the end of the launch (or
// when it is being aborted: q.stop).  Run by one whole wave; like next_task,
// no lane-dependent branch leaves its loop.
__device__ __forceinline__ uint32_t queue_next(const ExecParams& P, QueueState& q, uint32_t lane) {
  if (q.local != kExit) {
    const uint32_t pos = q.local;
    q.local = kExit;
    queue_progress(P, q, lane);
    return pos;
  }
  if (q.tile_i == q.tile_n) {
    uint32_t h = 0;
    if (lane == 0) h = __hip_atomic_fetch_add(q_head(P, q.shard), P.qtile, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    q.tile_h = rl(h, 0);
    q.tile_n = P.qtile;
    q.tile_i = 0;
  }
  const uint32_t t = q.tile_h + q.tile_i;
  if (t >= P.qcap) {  // beyond every sentinel: the protocol's bound was broken
    q.stop = kStuck;
    q.stuck = t;
    return kExit;
  }
  const uint32_t* slot = P.q + (size_t)q.shard * P.qcap + t;
  uint32_t v = uni(ld_coherent(slot));
  if (v == kQEmpty) {
    queue_report(P, q, lane);  // nothing to run now: report the finished sinks first
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    // a fixed back-off here, not the growing one of the lists: a queue
    // worker waits for whichever task is pushed next, and in the serving
    // loop a late claim delays a request (median latency 9.7 ms with the
    // fixed back-off, 11.4 ms with the growing one, same box).  Four naps (0.2
    // us) a poll for the first 64 (stencil 1024 x 500 1.76 ms, with one nap 1.80,
    // with 16 1.83), then the configured number
    __builtin_amdgcn_s_setprio(kPrioPoll);
    for (uint32_t spins = 1;; ++spins) {
      const uint32_t nap = spins < 64 ? 4u : P.idle_sleep;
      for (uint32_t i = 0; i < nap; ++i) __builtin_amdgcn_s_sleep(2);
      v = uni(ld_coherent(slot));
      if (v != kQEmpty) break;
      if ((spins & 63u) == 0u) {
        if (uni(ld_coherent(&P.ctrl->abort)) != 0u) return kExit;
        if (stalled(P, t0, __builtin_amdgcn_s_memrealtime()) || (P.spin_limit != 0u && spins >= P.spin_limit)) {
          q.stop = kStuck;
          q.stuck = t;
          return kExit;
        }
      }
    }
    __builtin_amdgcn_s_setprio(kPrioShort);
  }
  ++q.tile_i;
  if (v == kQExit) return kExit;
  queue_progress(P, q, lane);
  return v;
}

// One wave's part of a completion: `ready` marks the lanes whose decrement
// emptied the counter of `dst`.  The scheduling wave (keep) holds on to the
// first of them when it has no next task yet; the rest are pushed into the
// next shard in turn with one atomic on its tail.
__device__ __forceinline__ void queue_push(const ExecParams& P, QueueState& q, bool keep, uint32_t lane, bool ready,
                                           uint32_t dst) {
  uint64_t m = uni64(__ballot(ready));
  if (!m) return;
  if (keep && q.local == kExit) {
    const uint32_t first = (uint32_t)__builtin_ctzll(m);
    q.local = __builtin_amdgcn_readlane(dst, first);
    m &= m - 1;
    if (lane == first) ready = false;
    if (!m) return;
  }
  const uint32_t s = q.pshard;
  q.pshard = (q.pshard + 1u) & (P.qshards - 1u);
  const uint32_t leader = (uint32_t)__builtin_ctzll(m);
  uint32_t base = 0;
  if (lane == leader)
    base = __hip_atomic_fetch_add(q_tail(P, s), (uint32_t)__builtin_popcountll(m), __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
  base = __builtin_amdgcn_readlane(base, leader);
  if (ready) {
    const uint32_t idx = base + (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1ull));
    if (idx < P.qcap) st_coherent(P.q + (size_t)s * P.qcap + idx, dst);
  }
  // a shard holds at most every task once plus the sentinels, so a full
  // shard means a broken protocol: stop the launch rather than lose a task
  if (base + (uint32_t)__builtin_popcountll(m) > P.qcap) queue_abort(P, q, lane, base);
}

// COMPLETED_EDGE for every out-edge, then the pushes (one per wave with
// ready successors).  The payload stores are drained first, as in the list
// dispatch.
template <class Team>
__device__ __forceinline__ void complete_edges_q(const Team& tm, const ExecParams& P, const Rec& r, QueueState& q,
                                                 bool keep) {
  vm_drain();
  tm.sync();
  const uint32_t lane = tm.t & 63u;
  for (uint32_t j0 = 0; j0 < r.nsucc; j0 += tm.size()) {
    const uint32_t j = j0 + tm.t;
    bool ready = false;
    uint32_t dst = 0;
    if (j < r.nsucc) {
      dst = j0 == 0 ? r.succ0 : P.succ_pos[r.succ_beg + j];
      ready = __hip_atomic_fetch_sub(P.cnt + dst, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 1u;
    }
    queue_push(P, q, keep, lane, ready, dst);
  }
}

// Per-graph completion (launches that report graphs as they finish): a
// finished sink adds one to its graph's count; the addition that completes
// it stores the launch's sequence number into the graph's flag in host
// memory.  Every task of the graph precedes one of its sinks, and every
// sink's stores were drained before its addition, so the graph's results are
// in memory when the flag is seen.
__device__ __forceinline__ void graph_sink_done(const ExecParams& P, uint32_t graph, bool lead) {
  if (!P.gdone || !lead) return;
  const uint32_t old = __hip_atomic_fetch_add(P.gdone + graph, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (old + 1u == as_const(P.gtab)[graph].nsinks)
    __hip_atomic_store(P.gflag + graph, P.gseq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// With per-graph completion a digest is stored before the store drain, so that
// a graph's digests are in memory once its last sink has been counted; else
// after the edge signals, which do not wait for its reduction then (random
// pattern 1024 x 50: 242 against 258 us).
template <bool FULL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_exec_wave_q(ExecParams P) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t worker = uni((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  if (worker >= P.nworkers || gate_closed(P)) return;
  const WaveTeam tm{lane};
  if (FULL && P.diag && lane == 0)
    __hip_atomic_fetch_add(&P.ctrl->started, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  QueueState q;
  queue_init(q, P, worker);
  for (;;) {
    const uint32_t pos = queue_next(P, q, lane);
    if (pos == kExit) break;
    Rec r;
    unpack_rec(tm, P, rec_dword(P, pos, lane), r);
    const uint32_t part = run_body<FULL>(tm, P, pos, r, NoPrefetch());
    if (P.gdone) store_digest(tm, r, part);
    if (r.nsucc == 0u) ++q.sinks;
    complete_edges_q(tm, P, r, q, true);
    if (!P.gdone) store_digest(tm, r, part);
    if (r.nsucc == 0u) graph_sink_done(P, r.graph, lane == 0);
    if (FULL && P.tstamp && lane == 0) P.tstamp[2 * pos + 1] = __builtin_amdgcn_s_memrealtime();
  }
  if (q.stop == kStuck) queue_abort(P, q, lane, q.stuck);
}

// One workgroup per task: wave 0 takes the tasks and stages the record in
// LDS; every wave pushes the successors its lanes made ready.
template <bool FULL>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_exec_block_q(ExecParams P) {
  __shared__ uint32_t lds[32];
  __shared__ uint32_t cmd;
  __shared__ uint32_t recl[32];
  const uint32_t worker = blockIdx.x;
  if (worker >= P.nworkers || gate_closed(P)) return;
  const BlockTeam tm{threadIdx.x, blockDim.x, lds};
  const uint32_t lane = threadIdx.x & 63u, wave = uni(threadIdx.x >> 6);
  if (FULL && P.diag && threadIdx.x == 0)
    __hip_atomic_fetch_add(&P.ctrl->started, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  QueueState q;
  queue_init(q, P, worker);
  for (;;) {
    if (wave == 0) {
      const uint32_t pos = queue_next(P, q, lane);
      if (pos != kExit && lane < 32) recl[lane] = rec_dword(P, pos, lane);
      if (lane == 0) cmd = pos;
    }
    __syncthreads();
    const uint32_t pos = uni(cmd);
    const uint32_t v = recl[lane & 31u];
    __syncthreads();
    if (pos == kExit) break;
    Rec r;
    unpack_rec(tm, P, v, r);
    const uint32_t part = run_body<FULL>(tm, P, pos, r, NoPrefetch());
    if (P.gdone) store_digest(tm, r, part);
    if (wave == 0 && r.nsucc == 0u) ++q.sinks;
    complete_edges_q(tm, P, r, q, wave == 0);
    if (!P.gdone) store_digest(tm, r, part);
    if (r.nsucc == 0u) graph_sink_done(P, r.graph, threadIdx.x == 0);
    if (FULL && P.tstamp && threadIdx.x == 0) P.tstamp[2 * pos + 1] = __builtin_amdgcn_s_memrealtime();
    __syncthreads();
  }
  if (wave == 0 && q.stop == kStuck) queue_abort(P, q, lane, q.stuck);
}

// Empties the slots the previous launch filled: [0, tail) of every shard.
__global__ __launch_bounds__(256) void k_queue_clear(ExecParams P) {
  const uint32_t stride = gridDim.x * blockDim.x;
  for (uint32_t s = 0; s < P.qshards; ++s) {
    uint32_t t = *q_tail(P, s);
    if (t > P.qcap) t = P.qcap;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < t; i += stride) P.q[(size_t)s * P.qcap + i] = kQEmpty;
  }
}

// Residency probes: the executors' launch bounds and occupancy attributes
// (so the same number of blocks fits per CU), kept as kernels of their own so
// that kernel traces of real launches are not mixed with probe launches.
// Every wave of a block stays until the probe is over, so a probe block
// occupies what an executor block occupies.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_probe_wave(ExecParams P) {
  const uint32_t worker = uni((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  if (worker >= P.nworkers) return;
  residency_probe(P, (threadIdx.x & 63u) == 0);
}

__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_probe_block(ExecParams P) {
  if (blockIdx.x >= P.nworkers) return;
  if (threadIdx.x < 64) residency_probe(P, threadIdx.x == 0);
  __syncthreads();
}

// Everything a launch starts from, in one kernel (a launch of its own costs
// about 10 us before the executor can start): counters, diagnostics, the shared
// arrays of implicit graphs, and the queue.
__global__ __launch_bounds__(256) void k_reset(ExecParams P) {
  const uint32_t stride = gridDim.x * blockDim.x;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < P.npos; i += stride) {
    P.cnt[i] = P.indeg[i];
    if (P.execs) P.execs[i] = 0;
  }
  for (uint64_t i = blockIdx.x * blockDim.x + threadIdx.x; i < P.data_words; i += stride) {
    uint32_t lo = 0, hi = P.ngraphs;  // the last graph whose words begin at or before i
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (P.gtab[mid].first <= i) lo = mid;
      else hi = mid;
    }
    const GraphEnt& g = P.gtab[lo];
    g.data[i - g.first] = h32k(g.key2, i - g.first);
  }
  // gangs add their members' digest parts into the digest words
  if (P.gang > 1)
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < P.npos; i += stride) {
      const uint32_t* rd = reinterpret_cast<const uint32_t*>(P.rec + i);
      P.gtab[rd[kDwGraph]].digest[rd[kDwTid]] = 0;
    }
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < P.nworkers; i += stride) {
    P.bell[i * kBellStride] = 0;
    if (P.wprog) P.wprog[i] = 0xFFFFFFFFu;
    if (P.wstamp)
      for (int k = 0; k < 4; ++k) P.wstamp[4 * i + k] = 0;
  }
  if (P.tstamp)
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < 2 * P.npos; i += stride) P.tstamp[i] = 0;
  // an abort of an earlier, not yet inspected launch stays visible
  if (blockIdx.x == 0 && threadIdx.x == 0) P.ctrl->sticky += P.ctrl->abort;
  __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x < 8) (&P.ctrl->abort)[threadIdx.x] = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    P.ctrl->progress = 0;
    P.ctrl->precond = 0;
  }
  if (!P.q) return;
  // queue: the sources dealt round-robin over the shards, and the rest of the
  // slots the previous launch filled emptied (the tails are still that
  // launch's); the last block to get there resets the heads, the tails and the
  // sink count, which every block has read by then
  const uint32_t S = P.qshards;
  for (uint32_t s = 0; s < S; ++s) {
    const uint32_t mine = (P.nsrc + S - 1u - s) / S, used = max(mine, min(*q_tail(P, s), P.qcap));
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < used; i += stride)
      P.q[(size_t)s * P.qcap + i] = i < mine ? P.qsrc[i * S + s] : kQEmpty;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  const uint32_t before = __hip_atomic_fetch_add(q_sinks(P) + 1, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
  if (before + 1u != gridDim.x) return;
  for (uint32_t s = 0; s < S; ++s) {
    *q_head(P, s) = 0u;
    *q_tail(P, s) = (P.nsrc + S - 1u - s) / S;
  }
  q_sinks(P)[0] = 0u;
  q_sinks(P)[1] = 0u;
}

// Comparator: one launch runs one task; ordering comes from the stream or
// from the hipGraph's dependency edges, so no counter is touched.
__global__ __launch_bounds__(64) void k_one_task(ExecParams P, uint32_t pos) {
  const WaveTeam tm{threadIdx.x};
  Rec r;
  unpack_rec(tm, P, rec_dword(P, pos, threadIdx.x), r);
  const uint32_t part = run_body<false>(tm, P, pos, r, NoPrefetch());
  store_digest(tm, r, part);
}

// -------------------------------------------- records built on the device

// Last graph whose `field` is <= x (the table ascends in it; graphs without
// tasks share their successor's base, so the last such graph is the one that
// holds x).
template <uint32_t GraphSrc::*F>
__device__ __forceinline__ uint32_t graph_of(const GraphSrc* g, uint32_t ng, uint32_t x) {
  uint32_t lo = 0, hi = ng;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (g[mid].*F <= x) lo = mid;
    else hi = mid;
  }
  return lo;
}

// One thread per position: the record of the task at that position (layout
// order = graph order, task ids ascending), its slices of the predecessor
// address and successor position arrays, and its counter reset value; then
// one thread per source: the launch's source list.
__global__ __launch_bounds__(256) void k_build_records(const GraphSrc* gsrc, uint32_t ng, uint32_t npos, uint32_t nsrc,
                                                       TaskRec* rec, uint64_t* pred_addr, uint32_t* succ_pos,
                                                       uint32_t* indeg, uint32_t* src) {
  const uint32_t stride = gridDim.x * blockDim.x;
  for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < npos; p += stride) {
    const uint32_t gi = graph_of<&GraphSrc::pos_base>(gsrc, ng, p);
    const GraphSrc& g = gsrc[gi];
    const uint32_t v = p - g.pos_base;
    TaskRec r;
    memset(&r, 0, sizeof(r));
    r.tid = v;
    r.graph = gi;
    r.rounds = g.rounds[v];
    r.shape = task_shape(g.mode, g.mode == 1 ? g.n : 0u);
    const uint64_t wbytes = (uint64_t)g.n * 4u;
    // the inline lists are filled with constant indices so that the record
    // stays in registers (a variable index would put it in scratch memory)
    if (g.mode == 1) {
      r.out = g.payload + (uint64_t)(g.slot ? g.slot[v] : v) * wbytes;
      const uint32_t d0 = g.pred_ptr[v], d1 = g.pred_ptr[v + 1];
      r.npred = d1 - d0;
      r.pred_beg = g.pred_base + d0;
#pragma unroll
      for (uint32_t k = 0; k < kInPred; ++k)
        if (k < r.npred) {
          const uint32_t q = g.preds[d0 + k];
          r.pred[k] = g.payload + (uint64_t)(g.slot ? g.slot[q] : q) * wbytes;
        }
      for (uint32_t j = d0; j < d1; ++j) {
        const uint32_t q = g.preds[j];
        pred_addr[g.pred_base + j] = g.payload + (uint64_t)(g.slot ? g.slot[q] : q) * wbytes;
      }
    } else {
      const uint32_t a0 = g.req_ptr[v];
      r.out = (uint64_t)(g.reqs + a0);
      r.nreq = g.req_ptr[v + 1] - a0;
    }
    const uint32_t s0 = g.succ_ptr[v], s1 = g.succ_ptr[v + 1];
    r.nsucc = s1 - s0;
    r.succ_beg = g.succ_base + s0;
#pragma unroll
    for (uint32_t k = 0; k < kInSucc; ++k)
      if (k < r.nsucc) r.succ[k] = g.pos_base + g.succ[s0 + k];
    for (uint32_t j = s0; j < s1; ++j) succ_pos[g.succ_base + j] = g.pos_base + g.succ[j];
    rec[p] = r;
    indeg[p] = g.indeg[v];
  }
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nsrc; i += stride) {
    const GraphSrc& g = gsrc[graph_of<&GraphSrc::src_base>(gsrc, ng, i)];
    src[i] = g.pos_base + g.src[i - g.src_base];
  }
}

// Pre-condition vertices met by the host or by another launch (Section 4.1):
// lane i polls flag i (system-scope loads of pinned host memory) until every
// flag holds at least its value, or gives up after timeout_ticks.
__global__ __launch_bounds__(64) void k_wait_flags(FlagWait fw, Ctrl* ctrl, uint32_t* alarm,
                                                   uint64_t timeout_ticks) {
  const uint32_t lane = threadIdx.x;
  const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
  for (;;) {
    bool met = true;
    if (lane < fw.n) met = __hip_atomic_load(fw.addr[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) >= fw.value[lane];
    const uint64_t unmet = __ballot(!met);
    if (unmet == 0ull) return;
    if (__builtin_amdgcn_s_memrealtime() - t0 > timeout_ticks) {
      if (lane == 0) {
        st_coherent(&ctrl->precond, 1u + (uint32_t)__builtin_ctzll(unmet));
        __hip_atomic_fetch_add(&ctrl->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        raise_alarm(alarm);
      }
      return;
    }
    __builtin_amdgcn_s_sleep(32);
  }
}

// Post-condition vertex: runs after the launch in stream order, so every
// task of it has finished; publishes them (system-scope release) and sets the
// flag, unless the launch was abandoned.
__global__ __launch_bounds__(64) void k_set_flag(uint32_t* flag, uint32_t value, const Ctrl* ctrl) {
  if (threadIdx.x != 0) return;
  if (__hip_atomic_load(&ctrl->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) return;
  __hip_atomic_store(flag, value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(256) void k_fill(uint32_t* p, uint64_t n, uint32_t v) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

// ---------------------------------------------------------------- launchers

hipError_t launch_build_records(const GraphSrc* gsrc, uint32_t ng, uint32_t npos, uint32_t nsrc, TaskRec* rec,
                                uint64_t* pred_addr, uint32_t* succ_pos, uint32_t* indeg, uint32_t* src,
                                hipStream_t s) {
  const uint32_t n = npos > nsrc ? npos : nsrc;
  uint32_t blocks = (n + 255u) / 256u;
  if (blocks > 8192u) blocks = 8192u;
  if (blocks == 0) blocks = 1;
  hipLaunchKernelGGL(k_build_records, dim3(blocks), dim3(256), 0, s, gsrc, ng, npos, nsrc, rec, pred_addr, succ_pos,
                     indeg, src);
  return hipGetLastError();
}

hipError_t launch_fill(uint32_t* p, uint64_t n, uint32_t v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  uint64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_fill, dim3((uint32_t)blocks), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}


hipError_t launch_wait_flags(const FlagWait& fw, Ctrl* ctrl, uint32_t* alarm, uint64_t timeout_ticks, hipStream_t s) {
  if (fw.n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_wait_flags, dim3(1), dim3(64), 0, s, fw, ctrl, alarm, timeout_ticks);
  return hipGetLastError();
}

hipError_t launch_set_flag(uint32_t* flag, uint32_t value, const Ctrl* ctrl, hipStream_t s) {
  hipLaunchKernelGGL(k_set_flag, dim3(1), dim3(64), 0, s, flag, value, ctrl);
  return hipGetLastError();
}

// A queue's blocks take a ticket each, so there are fewer of them.
hipError_t launch_reset(const ExecParams& p, hipStream_t s) {
  const uint64_t blocks = (std::max<uint64_t>(p.npos, p.data_words) + 255u) / 256u;
  const uint64_t most = p.q ? 1024u : 4096u;
  hipLaunchKernelGGL(k_reset, dim3((uint32_t)std::max<uint64_t>(1u, std::min(blocks, most))), dim3(256), 0, s, p);
  return hipGetLastError();
}

// The kernels come in two forms: with doorbells or diagnostics, and without.
hipError_t launch_exec(const ExecParams& p, uint32_t mapping, uint32_t wg_waves, uint32_t grid_blocks,
                       hipStream_t s) {
  const bool full = p.notify || p.diag;
  const dim3 grid(grid_blocks), wave(256), block(wg_waves * 64u);
  if (p.residency_probe) {
    if (mapping == 1) hipLaunchKernelGGL(k_probe_wave, grid, wave, 0, s, p);
    else hipLaunchKernelGGL(k_probe_block, grid, block, 0, s, p);
  } else if (mapping == 1) {
    if (full) hipLaunchKernelGGL(k_exec_wave<true>, grid, wave, 0, s, p);
    else hipLaunchKernelGGL(k_exec_wave<false>, grid, wave, 0, s, p);
  } else if (mapping == 2) {
    if (full) hipLaunchKernelGGL(k_exec_block<true>, grid, block, 0, s, p);
    else hipLaunchKernelGGL(k_exec_block<false>, grid, block, 0, s, p);
  } else {
    if (full) hipLaunchKernelGGL(k_exec_gang<true>, grid, block, 0, s, p);
    else hipLaunchKernelGGL(k_exec_gang<false>, grid, block, 0, s, p);
  }
  return hipGetLastError();
}

hipError_t launch_queue_clear(const ExecParams& p, hipStream_t s) {
  uint32_t blocks = (p.qcap + 255u) / 256u;
  if (blocks > 4096u) blocks = 4096u;
  if (blocks == 0) blocks = 1;
  hipLaunchKernelGGL(k_queue_clear, dim3(blocks), dim3(256), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_exec_queue(const ExecParams& p, uint32_t mapping, uint32_t wg_waves, uint32_t grid_blocks,
                             hipStream_t s) {
  const dim3 grid(grid_blocks), wave(256), block(wg_waves * 64u);
  if (mapping == 1) {
    if (p.diag) hipLaunchKernelGGL(k_exec_wave_q<true>, grid, wave, 0, s, p);
    else hipLaunchKernelGGL(k_exec_wave_q<false>, grid, wave, 0, s, p);
  } else {
    if (p.diag) hipLaunchKernelGGL(k_exec_block_q<true>, grid, block, 0, s, p);
    else hipLaunchKernelGGL(k_exec_block_q<false>, grid, block, 0, s, p);
  }
  return hipGetLastError();
}

int exec_blocks_per_cu(uint32_t mapping, uint32_t wg_waves) {
  int nb = 0;
  hipError_t e;
  // (both forms are held to eight wavefronts a SIMD)
  if (mapping == 1) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_exec_wave<true>, 256, 0);
  else e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_exec_block<true>, (int)(wg_waves * 64u), 0);
  if (e != hipSuccess) return -1;
  return nb;
}

hipError_t launch_one_task(const ExecParams& p, uint32_t pos, hipStream_t s) {
  hipLaunchKernelGGL(k_one_task, dim3(1), dim3(64), 0, s, p, pos);
  return hipGetLastError();
}

const void* one_task_kernel() { return (const void*)k_one_task; }

}  // namespace tg
