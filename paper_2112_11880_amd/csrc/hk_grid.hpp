// hk_grid.hpp -- grid-wide barrier for the persistent batched solvers.
//
// The persistent kernels are launched cooperatively (every workgroup
// resident), so a barrier cannot deadlock on scheduling.  The barrier is a
// flag array: each workgroup publishes the barrier's epoch in its own word
// (after a release fence for the data it wrote), workgroup 0 waits until
// every word shows the epoch, runs a callback (the second stage of the
// reductions and the per-system scalar updates), then publishes the epoch in
// a release word that the other workgroups wait on.  A single shared counter
// incremented by every workgroup cost ~136 us per barrier on MI355X (256
// serialised device-scope atomics); flags in separate words cost a few
// round trips.
//
// Only thread 0 of a workgroup fences; the workgroup barrier that follows
// orders the other threads after it (the usual grid-sync pattern).  On
// gfx950 an agent-scope acquire fence invalidates caches, and executing it in
// all 16 waves of a 1024-thread workgroup made one barrier cost ~63 us (one
// wave: a few us).  Each fence is one-sided: a release (L2 write-back) before
// a flag is published, an acquire (L2 invalidate) after one is observed.
// Two-sided fences at both points cost ~25 us more per solver iteration
// (5 barriers) on MI355X.
//
// Every wait has a time limit: a workgroup that waits longer than the
// barrier's spin_limit (kSpinLimitTicks unless the host sets another) raises
// an abort flag and every workgroup leaves the kernel at its next barrier,
// so a broken launch ends instead of hanging.
#pragma once

#include <cstdlib>

#include "hk_common.hpp"

namespace hk {

constexpr int kBarMaxBlocks = 1024;

struct GridBar {
  unsigned release;      // last epoch released by workgroup 0
  int abort;
  unsigned long long spin_limit;  // wall-clock ticks a wait may take before it aborts
  // optional: stamps[e] = wall clock (100 MHz ticks) when every workgroup had
  // arrived at barrier e, for e < nstamps (null: none)
  double* stamps;
  unsigned long long nstamps;
  // per-XCD-group sums of barrier_reduce: kXcds x 4 x 64 doubles (null if unused)
  double* gpart;
  unsigned pad[54];      // keep release/abort on their own 256-byte line
  unsigned arrive[kBarMaxBlocks];  // last epoch each workgroup arrived at
  unsigned garrive[kXcds];         // last epoch each group's sums were published at
};

// 100 MHz constant clock: 4e8 ticks = 4 s.
constexpr unsigned long long kSpinLimitTicks = 400000000ull;

__device__ __forceinline__ unsigned ld_relaxed_u32(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int ld_relaxed_i32(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_relaxed_u32(unsigned* p, unsigned v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits (one thread) until *p >= e; false on abort or time-out (which raises abort).
__device__ __forceinline__ bool wait_epoch(const unsigned* p, unsigned e, GridBar* bar) {
  const unsigned long long t0 = wall_clock64();
  const unsigned long long limit = bar->spin_limit;
  while (ld_relaxed_u32(p) < e) {
    __builtin_amdgcn_s_sleep(1);
    if (ld_relaxed_i32(&bar->abort)) return false;
    if (wall_clock64() - t0 > limit) {
      atomicExch(&bar->abort, 1);
      return false;
    }
  }
  return true;
}

// Grid barrier; on_last() runs in workgroup 0 (all its threads) once every
// workgroup has arrived.  `epoch` is the caller's per-workgroup counter
// (start at 0; the barrier memory must be zeroed before the launch).
// Returns true if the kernel must stop (abort raised somewhere).  All
// threads of every workgroup must call it.
template <class F>
__device__ __forceinline__ bool barrier_last(GridBar* bar, unsigned& epoch, F&& on_last) {
  __shared__ int s_stop;
  const unsigned e = ++epoch;
  __syncthreads();
  if (threadIdx.x == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");  // this workgroup's writes before its flag
    st_relaxed_u32(&bar->arrive[blockIdx.x], e);
  }
  if (blockIdx.x == 0) {
    bool ok = true;
    for (int b = threadIdx.x; b < (int)gridDim.x; b += blockDim.x) ok = wait_epoch(&bar->arrive[b], e, bar) && ok;
    if (!ok) atomicExch(&bar->abort, 1);
    __syncthreads();
    if (threadIdx.x == 0) {
      s_stop = ld_relaxed_i32(&bar->abort);
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // every workgroup's writes
      if (bar->stamps && e < bar->nstamps) bar->stamps[e] = (double)wall_clock64();
    }
    __syncthreads();
    if (!s_stop) on_last();
    __syncthreads();
    if (threadIdx.x == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");  // the callback's writes before the epoch
      st_relaxed_u32(&bar->release, e);
    }
  } else if (threadIdx.x == 0) {
    (void)wait_epoch(&bar->release, e, bar);
  }
  if (threadIdx.x == 0) {
    s_stop = ld_relaxed_i32(&bar->abort);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // workgroup 0's release, and through it every arrival
  }
  __syncthreads();
  return s_stop != 0;
}

// ------------------------------------------------- barrier that sums to all
//
// The resident solvers' barrier: every workgroup publishes its NV partial
// sums as 8-byte words and reads every workgroup's words itself, so one trip
// through memory is both the barrier and the reduction, and every workgroup
// holds the totals (summed in one order, so the same bits everywhere).  On
// MI355X it takes 1.9 us with 20 workgroups, 2.3 with 64 and 4 with 256
// (three sums), against 9.4 us for the flag barrier above with its release
// fence, workgroup 0's callback and the second trip.
//
//  - A word is its own flag: kSumEmpty, a NaN no sum is published as, means
//    "not there yet".  A workgroup that has seen every word of epoch e knows
//    that all have finished reading epoch e - 1 and empties its own words of
//    that epoch; with kSumSets sets in turn they are used again at e + 3.
//  - A workgroup's words lie together, so that one 16-byte store or load
//    moves two of them (each word is still a flag of its own: nothing relies
//    on the two arriving together).  With three sums a word each, the barrier
//    took 1.4 us longer at 256 workgroups than with one.
//  - The words are published kSumReps times and a workgroup reads copy
//    rank % kSumReps: 256 workgroups polling one copy slow the stores to it
//    (64 workgroups: 3.2 us with one copy, 2.4 with eight).
//  - No release fence: what the other workgroups read (publish below) is
//    stored past the L2 at agent scope, and every wave waits for its stores
//    before the words are published.  The plain-store form with an L2
//    write-back took 13-17 us per barrier and gather at 256 workgroups,
//    against 7.5-10.
//  - The acquire (an L1 and L2 invalidate, 1.1 us at 256 workgroups) is thread
//    0's alone, as above, and only where the caller asks for it: it has to
//    drop the lines of a published vector's previous contents, so one between
//    the last reads of a vector's contents and the first reads of the next
//    ones at the same addresses is enough, and vectors published to kRing
//    places in turn need one every kRing times (see hk_resident.hpp).  It may
//    run before another workgroup has arrived: a vector is stored only after
//    a barrier that follows the last reads of what it overwrites.
constexpr int kSumSets = 4;
constexpr int kSumReps = 8;
constexpr int kSumWords = 4;    // at most this many sums
constexpr int kSumBlocks = 256; // at most this many workgroups
constexpr size_t kSumSetWords = (size_t)kSumReps * kSumWords * kSumBlocks;
constexpr unsigned long long kSumEmpty = 0x7ff8dead0000beefull;

struct GridSum {
  unsigned long long* words;      // kSumSets * kSumSetWords, all kSumEmpty at launch
  int* abort;                     // 0 at launch
  unsigned long long spin_limit;  // wall-clock ticks a wait may take before it aborts
  // The workgroups share an XCD and with it the L2: what they publish need not
  // go past it (0 at launch; set by the kernel, in all of them alike, from
  // what same_xcd_sums has summed).  A load at agent scope passes by the L1 only
  // where the line is in the L2, so the polling is the same.  Barrier, one
  // published vector and four gathers: 3.1 -> 1.6 us for 20 workgroups, 3.3 -> 1.7
  // for 32.
  int local;
};

__device__ __forceinline__ void st_agent_u64(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Agent-scope (sc1) accesses of 16 bytes have no form in the language; these
// use the buffer instructions' builtins.  (In inline asm the compiler keeps
// none of the wait states that a store's scalar base and data registers need
// around it.)
typedef int ni4 __attribute__((ext_vector_type(4)));
typedef int ni2 __attribute__((ext_vector_type(2)));
typedef unsigned long long nu2 __attribute__((ext_vector_type(2)));
constexpr int kAuxSc1 = 16;
template <class V> __device__ __forceinline__ __amdgpu_buffer_rsrc_t pub_rsrc(V* p) {
  // raw buffer over the whole 32-bit offset range; the offsets used are those
  // of elements of p
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)0xffffffffu, 0x00020000);
}

// 16 bytes at byte offset `off` of p for the other workgroups.
template <class T> __device__ __forceinline__ void store_shared(const GridSum& gs, T* p, int off, ni4 q) {
  if (gs.local) __builtin_amdgcn_raw_buffer_store_b128(q, pub_rsrc(p), off, 0, 0);
  else __builtin_amdgcn_raw_buffer_store_b128(q, pub_rsrc(p), off, 0, kAuxSc1);
}
// Stores element i of a vector that other workgroups read after the next
// barrier.
__device__ __forceinline__ void publish(const GridSum& gs, double2* p, unsigned i, double2 v) {
  const nd2 q = {v.x, v.y};
  store_shared(gs, p, (int)(i * (unsigned)sizeof(v)), __builtin_bit_cast(ni4, q));
}
__device__ __forceinline__ void publish(const GridSum& gs, float2* p, unsigned i, float2 v) {
  const nf2 q = {v.x, v.y};
  const int off = (int)(i * (unsigned)sizeof(v));
  if (gs.local) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(ni2, q), pub_rsrc(p), off, 0, 0);
  else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(ni2, q), pub_rsrc(p), off, 0, kAuxSc1);
}

// Two sums over the workgroups (one thread of each adds to them) that tell
// whether all run on one XCD; same_xcd reads the totals.
__device__ __forceinline__ void same_xcd_sums(double& s1, double& s2) {
  if (threadIdx.x != 0) return;
  const double x = (double)__builtin_amdgcn_s_getreg(20 | (3 << 11));  // XCC_ID, 4 bits
  s1 = x;
  s2 = x * x;
}
__device__ __forceinline__ int same_xcd(int size, double s1, double s2) {
  return __builtin_amdgcn_readfirstlane((int)((double)size * s2 == s1 * s1));
}

// v + (v of the lane the DPP control names; 0 where there is none)
template <int CTRL> __device__ __forceinline__ double dpp_add(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
  return v + __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// Sum over the wave, valid in lane 63: shifts by 1, 2, 4, 8 within the rows
// of 16 lanes, then row totals passed on (row_bcast 15 and 31).
__device__ __forceinline__ double wave_sum63(double v) {
  v = dpp_add<0x111>(v);
  v = dpp_add<0x112>(v);
  v = dpp_add<0x114>(v);
  v = dpp_add<0x118>(v);
  v = dpp_add<0x142>(v);
  return dpp_add<0x143>(v);
}
// A sum as a word: any NaN as the one quiet NaN, never as kSumEmpty.
__device__ __forceinline__ unsigned long long sum_word(double s) {
  return s == s ? (unsigned long long)__double_as_longlong(s) : 0x7ff8000000000000ull;
}
// (threads that wait) whether to give up: past the limit this thread raises
// the flag, and now and then looks whether another has.
__device__ __forceinline__ bool sum_give_up(const GridSum& gs, unsigned long long t0, int spins) {
  const bool late = wall_clock64() - t0 > gs.spin_limit;
  if (late) atomicExch(gs.abort, 1);
  return (late || (spins & 15) == 15) && ld_relaxed_i32(gs.abort) != 0;
}

// One barrier of `size` <= kSumBlocks workgroups of NT threads, the caller's
// being number `rank` of them: v (each thread's partial sums) becomes the
// totals, in every thread.  `epoch` starts at 0.  lds: room for
// kSumWords * (NT / 64 + 4) doubles, used by nothing else.  With INV the
// caller's caches drop what they hold.  Returns true if the kernel must stop
// (a wait passed the limit here or elsewhere).  With `running` (a device count)
// the others may come late, each from work of its own: the limit then counts only
// while *running is 0.  All threads of the workgroups call it.
template <int NV, int NT>
__device__ __forceinline__ bool group_sum(const GridSum& gs, int size, int rank, unsigned& epoch, bool inv,
                                          double (&v)[NV], double* lds, const int* running = nullptr) {
  static_assert(NV >= 1 && NV <= kSumWords && NT >= kSumBlocks, "sums and pollers");
  constexpr int W = NT / kWave, NP = (NV + 1) / 2;  // pairs of words
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  double* totals = lds + kSumWords * W;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const double s = wave_sum63(v[k]);
    if (lane == kWave - 1) lds[k * W + w] = s;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's published elements
  __syncthreads();
  unsigned long long* set = gs.words + (epoch % kSumSets) * kSumSetWords;
  unsigned long long* old = gs.words + ((epoch + kSumSets - 1) % kSumSets) * kSumSetWords;
  // byte offset of copy `rep` of workgroup b's words
  auto at_word = [](int rep, int b) { return (rep * kSumBlocks + b) * (kSumWords * 8); };
  static_assert(kSumReps * kSumWords <= kWave, "one wave publishes");
  if (threadIdx.x < kSumReps * kSumWords) {
    const int k = threadIdx.x % kSumWords, rep = threadIdx.x / kSumWords;
    double s = 0;
    if (k < NV) {
#pragma unroll
      for (int j = 0; j < W; ++j) s += lds[k * W + j];
    }
    const unsigned long long mine = sum_word(s), next = __shfl_down(mine, 1);
    if (k % 2 == 0 && k < NV) {
      const nu2 pair = {mine, next};
      store_shared(gs, set, at_word(rep, rank) + k * 8, __builtin_bit_cast(ni4, pair));
    }
  }
  bool ok = true;
  double part[2 * NP];
#pragma unroll
  for (int k = 0; k < 2 * NP; ++k) part[k] = 0;
  if ((int)threadIdx.x < size) {
    const int off = at_word(rank % kSumReps, threadIdx.x);
    unsigned long long t0 = wall_clock64();
    nu2 q[NP];
    for (int spins = 0;; ++spins) {
      bool all = true;
      asm volatile("" ::: "memory");  // loaded anew in every turn
#pragma unroll
      for (int k = 0; k < NP; ++k)
        q[k] = __builtin_bit_cast(nu2, __builtin_amdgcn_raw_buffer_load_b128(pub_rsrc(set), off + 16 * k, 0, kAuxSc1));
#pragma unroll
      for (int k = 0; k < NV; ++k) all = all && q[k / 2][k % 2] != kSumEmpty;
      if (all) break;
      if (running && (spins & 15) == 14 && ld_relaxed_i32(running) > 0) t0 = wall_clock64();
      if (sum_give_up(gs, t0, spins)) { ok = false; break; }
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) part[k] = __longlong_as_double((long long)q[k / 2][k % 2]);
  }
  if (inv && threadIdx.x == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  if (w < kSumBlocks / kWave) {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const double s = wave_sum63(part[k]);
      if (lane == kWave - 1) totals[k * 4 + w] = s;
    }
  }
  const int stop = __syncthreads_or(!ok);
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    v[k] = totals[k * 4] + totals[k * 4 + 1] + totals[k * 4 + 2] + totals[k * 4 + 3];
  }
  if (threadIdx.x < 2 * kSumReps) {
    const nu2 empty = {kSumEmpty, kSumEmpty};
    store_shared(gs, old, at_word(threadIdx.x / 2, rank) + 16 * (threadIdx.x % 2), __builtin_bit_cast(ni4, empty));
  }
  ++epoch;
  return stop != 0;
}

// ------------------------------------------------ the same for many sums
//
// Up to kManySums sums in two trips: every workgroup publishes its partial
// sums, one wave somewhere in the grid adds each component over the
// workgroups and publishes the total (kSumReps copies), every workgroup
// reads the totals.  Two sets of partial words and kSumSets of totals are
// used in turn: a workgroup that has seen every total of one call knows that
// all partials of it have been read, and that everybody is past reading the
// totals of the call before.
constexpr int kManySums = 96;
constexpr size_t kManyPart = (size_t)kManySums * kSumBlocks;
constexpr size_t kManyTot = (size_t)kSumReps * kManySums;
constexpr size_t kManyWords = 2 * kManyPart + kSumSets * kManyTot;

// `waves`: the workgroup's partial sums by wave, waves[c * W + w] for c < nc,
// written before the call; totals[c] on return, in LDS.  `call` starts at 0.
// As group_sum without INV otherwise; all threads of every workgroup call it.
template <int NT>
__device__ __forceinline__ bool grid_sum_many(const GridSum& gs, int G, int rank, unsigned long long* many,
                                              unsigned& call, int nc, const double* waves, double* totals) {
  constexpr int W = NT / kWave;
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  unsigned long long* part = many + (call & 1) * kManyPart;
  unsigned long long* tot = many + 2 * kManyPart + (call % kSumSets) * kManyTot;
  unsigned long long* old = many + 2 * kManyPart + ((call + kSumSets - 1) % kSumSets) * kManyTot;
  const unsigned long long t0 = wall_clock64();
  auto st_word = [&](unsigned long long* p, unsigned long long v) {
    if (gs.local) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    else st_agent_u64(p, v);
  };
  bool ok = true;
  auto wait_word = [&](const unsigned long long* p) {
    unsigned long long q;
    for (int spins = 0;; ++spins) {
      q = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (q != kSumEmpty) break;
      if (sum_give_up(gs, t0, spins)) { ok = false; break; }
    }
    return __longlong_as_double((long long)q);
  };
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  for (int c = threadIdx.x; c < nc; c += NT) {
    double s = 0;
    for (int j = 0; j < W; ++j) s += waves[c * W + j];
    st_word(part + (size_t)c * kSumBlocks + rank, sum_word(s));
  }
  // the components this wave adds up
  for (int c = rank + G * w; c < nc; c += G * W) {
    // all of a lane's words in flight together
    const unsigned long long* pc = part + (size_t)c * kSumBlocks;
    constexpr int U = kSumBlocks / kWave;
    unsigned long long v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      v[u] = lane + u * kWave < G
                 ? __hip_atomic_load(pc + lane + u * kWave, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                 : 0ull;
    double s = 0;
#pragma unroll
    for (int u = 0; u < U; ++u)
      s += v[u] == kSumEmpty ? wait_word(pc + lane + u * kWave) : __longlong_as_double((long long)v[u]);
    s = wave_sum63(s);
    const unsigned long long q = __shfl(sum_word(s), kWave - 1);
    if (lane < kSumReps) st_word(tot + (size_t)lane * kManySums + c, q);
  }
  for (int c = threadIdx.x; c < nc; c += NT)
    totals[c] = wait_word(tot + (size_t)(rank % kSumReps) * kManySums + c);
  const int stop = __syncthreads_or(!ok);
  for (int c = threadIdx.x; c < nc; c += NT)
    st_word(part + (size_t)c * kSumBlocks + rank, kSumEmpty);
  if (call > 0)
    for (int c = rank + G * w; c < nc; c += G * W)
      if (lane < kSumReps) st_word(old + (size_t)lane * kManySums + c, kSumEmpty);
  ++call;
  return stop != 0;
}

// ---------------------------------------- the same for the sums of several solves
//
// Up to 2 NP sums.  A workgroup's words fill a row of 16 NP bytes, kWideReps
// times; the threads read all rows in order, 16 bytes a lane, each thread the
// same pair of sums of NT / NP rows apart, so that a wave is left with 64 / NP
// partial sums of a pair to add.  (group_sum gives a thread one workgroup's words
// and the wave a full reduction for every sum.)
constexpr int kWideReps = 4;

// a + (a of the other half) in the lower 32 lanes, the same of b in the upper;
// with HALF = 16 in the even and odd rows of 16 lanes: two values' sums step on
// in one register.
template <int HALF> __device__ __forceinline__ double fold(double a, double b) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(a), y = (unsigned long long)__double_as_longlong(b);
  unsigned r[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const unsigned u = (unsigned)(x >> (32 * h)), v = (unsigned)(y >> (32 * h));
    if constexpr (HALF == 32) {
      const auto t = __builtin_amdgcn_permlane32_swap(u, v, false, false);
      r[0][h] = t[0];
      r[1][h] = t[1];
    } else {
      const auto t = __builtin_amdgcn_permlane16_swap(u, v, false, false);
      r[0][h] = t[0];
      r[1][h] = t[1];
    }
  }
  return __longlong_as_double((long long)(((unsigned long long)r[0][1] << 32) | r[0][0])) +
         __longlong_as_double((long long)(((unsigned long long)r[1][1] << 32) | r[1][0]));
}
// Sums of four values over the wave, in lanes 15 (a), 31 (c), 47 (b) and 63 (d):
// 21 instructions where four wave_sum63 take 72.
__device__ __forceinline__ double wave_sums4(double a, double b, double c, double d) {
  double v = fold<16>(fold<32>(a, b), fold<32>(c, d));
  v = dpp_add<0x111>(v);
  v = dpp_add<0x112>(v);
  v = dpp_add<0x114>(v);
  return dpp_add<0x118>(v);
}
template <int NP> struct WideSum {
  static constexpr size_t kSetWords = (size_t)kWideReps * kSumBlocks * NP * 2;
  static constexpr size_t kWords = kSumSets * kSetWords;
};

// waves[c * W + w], c < nv: the workgroup's partial sums by wave, written before
// the call; parts[c * W + w] on return: partial totals, to be added over w.
// Otherwise as group_sum without INV.
template <int NP, int NT>
__device__ __forceinline__ bool group_sum_wide(const GridSum& gs, unsigned long long* words, int size, int rank,
                                               unsigned& epoch, int nv, const double* waves, double* parts) {
  constexpr int W = NT / kWave, kRows = NT / NP, U = (kSumBlocks + kRows - 1) / kRows;
  static_assert(kWideReps * NP <= NT && kWave % NP == 0, "one store per thread, pairs within a wave");
  const int np = (nv + 1) / 2;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // addresses are not worth registers from call to call
  const int pair = tid % NP;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's published elements
  __syncthreads();
  unsigned long long* set = words + (epoch % kSumSets) * WideSum<NP>::kSetWords;
  unsigned long long* old = words + ((epoch + kSumSets - 1) % kSumSets) * WideSum<NP>::kSetWords;
  auto at_pair = [&](int rep, int b) { return ((rep * kSumBlocks + b) * NP + pair) * 16; };
  if (tid < kWideReps * NP && pair < np) {
    double s[2] = {0, 0};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = 2 * pair + h;
      if (c < nv)
        for (int j = 0; j < W; ++j) s[h] += waves[c * W + j];
    }
    const nu2 mine = {sum_word(s[0]), sum_word(s[1])};
    store_shared(gs, set, at_pair(tid / NP, rank), __builtin_bit_cast(ni4, mine));
  }
  bool ok = true;
  double tot[2] = {0, 0};
  if (pair < np) {
    const int rep = rank % kWideReps, row = tid / NP;
    const unsigned long long t0 = wall_clock64();
    auto fetch = [&](int b) {
      return __builtin_bit_cast(nu2, __builtin_amdgcn_raw_buffer_load_b128(pub_rsrc(set), at_pair(rep, b), 0, kAuxSc1));
    };
    nu2 q[U];
    for (int spins = 0;; ++spins) {
      bool all = true;
      asm volatile("" ::: "memory");  // loaded anew in every turn
#pragma unroll
      for (int u = 0; u < U; ++u) q[u] = fetch(min(row + u * kRows, size - 1));
#pragma unroll
      for (int u = 0; u < U; ++u) all = all && q[u][0] != kSumEmpty && q[u][1] != kSumEmpty;
      if (all) break;
      if (sum_give_up(gs, t0, spins)) { ok = false; break; }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = row + u * kRows < size;
      tot[0] += in ? __longlong_as_double((long long)q[u][0]) : 0.0;
      tot[1] += in ? __longlong_as_double((long long)q[u][1]) : 0.0;
    }
  }
#pragma unroll
  for (int d = NP; d < kWave; d *= 2) {
    tot[0] += __shfl_xor(tot[0], d);
    tot[1] += __shfl_xor(tot[1], d);
  }
  if (tid % kWave < NP) {
    const int w = tid / kWave;
    parts[(2 * pair) * W + w] = tot[0];
    parts[(2 * pair + 1) * W + w] = tot[1];
  }
  const int stop = __syncthreads_or(!ok);
  if (tid < kWideReps * NP) {
    const nu2 empty = {kSumEmpty, kSumEmpty};
    store_shared(gs, old, at_pair(tid / NP, rank), __builtin_bit_cast(ni4, empty));
  }
  ++epoch;
  return stop != 0;
}

// Host: the spin limit of a launch, kSpinLimitTicks unless the environment
// variable HK_BARRIER_SPIN_TICKS holds a positive count (tests use a tiny
// one to drive the abort path).
inline unsigned long long barrier_spin_limit() {
  const char* v = getenv("HK_BARRIER_SPIN_TICKS");
  if (v) {
    const unsigned long long t = strtoull(v, nullptr, 10);
    if (t > 0) return t;
  }
  return kSpinLimitTicks;
}

}  // namespace hk
