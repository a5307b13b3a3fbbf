// hk_resident.hpp -- what the resident solves share (hk_resident.hip,
// hk_resident_l.hip): a thread's rows of the matrix, the launch.
#pragma once

#include <algorithm>
#include <vector>

#include "hk_grid.hpp"
#include "hk_internal.hpp"
#include "hk_solver.hpp"

namespace hk {

// Published vectors go to kRing places in turn, so that the caches have to be
// dropped (group_sum's argument) once in several publications only: content c
// is at place c % kRing, and takes the place of content c - kRing.  Wanted is
// one barrier that drops them, entered by every workgroup after the last reads
// of content c - kRing -- a barrier that those reads merely precede in their own
// workgroup is not enough, another one on the same L2 may still read -- and left
// before the first reads of content c.  Each kernel says which of its barriers
// these are.  Dropping them at every barrier cost 1.1 us of each at 256
// workgroups.
constexpr int kRing = 4;
constexpr int kSweepLanes = 64;  // columns of a sweep's right-hand sides
// Waves per SIMD that the single solves' kernels leave room for: two workgroups
// of 256 threads per CU, which a packed launch of up to 64 workgroups counts on
// (the compiler gives a 256-thread kernel more than 256 registers otherwise, and
// BiCGStab(l) took 261 and 274 for rows of 15 and 27 entries).
constexpr int kResWaves = 2;

template <class R> struct ResArgs {
  using V = cplx<R>;
  int n, rows;             // rows per workgroup: a multiple of 64
  int packed;              // the launch has kXcds times the workgroups: see ResPlace
  const int* rowptr;
  const int* col;
  const V* val;
  const V* dinv;
  const V* b;
  const V* x0;             // null: start from 0; else r0 holds b - A x0
  const V* r0;
  V* y;                    // D x at the end
  V* pub;                  // published vectors: vector i, place p at pub + (kRing i + p) stride
  long long stride;        // elements
  SolveState* st;          // the solve's state at the end
  const int* flag;         // zero-diagonal flag of the set-up: nonzero ends the kernel
  GridSum gs;
  double tol;
  long long maxit;
  double* history;
  // entry p of A, with column c: of Ahat; the right-hand side's row
  __device__ __forceinline__ V entry(int p) const { return val[p]; }
  __device__ __forceinline__ V scaled(int p, int c) const;
  __device__ __forceinline__ V rhs(int row) const { return b[row]; }
  __device__ __forceinline__ V inv_diag(int row) const { return dinv[row]; }
};

// ---------------------------------------------------------- device helpers

template <class R> __device__ __forceinline__ cplx<R> ResArgs<R>::scaled(int p, int c) const {
  return cmul(val[p], dinv[c]);
}

template <class V> struct Pair { V u, v; };

// acc - a * b, in explicit multiply-adds: a product's operand has the same bits
// where its owner and where another thread forms it.
template <class V> __device__ __forceinline__ V cfnma(V a, V b, V acc) {
  acc.x = fma(-a.x, b.x, fma(a.y, b.y, acc.x));
  acc.y = fma(-a.x, b.y, fma(-a.y, b.x, acc.y));
  return acc;
}

// A value every thread holds alike, moved to scalar registers (the vector
// ones are for the matrix).
__device__ __forceinline__ double uni(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readfirstlane((int)b), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double2 uni(double2 v) { return make_double2(uni(v.x), uni(v.y)); }
template <class T> __device__ __forceinline__ T* uni(T* p) {
  const unsigned long long b = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane((int)b), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return reinterpret_cast<T*>(((unsigned long long)hi << 32) | lo);
}

// Element of a published vector at byte offset `off`: a scalar base and a
// 32-bit lane offset.
template <class V> __device__ __forceinline__ V at(const V* base, unsigned off) {
  return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(base) + off);
}
// The column offset, hidden from loop-invariant code motion: otherwise the
// compiler keeps a 64-bit address per entry and vector in registers across
// iterations, three times what the entries themselves take.
__device__ __forceinline__ unsigned fresh(unsigned off) {
  asm volatile("" : "+v"(off));
  return off;
}

// v is computed before this point and later loads are issued after it (the
// compiler keeps loads in order with the clobber, and otherwise gathers all of
// them in front of the arithmetic).
template <class V> __device__ __forceinline__ void here(V& v) {
  asm volatile("" : "+v"(v.x), "+v"(v.y)::"memory");
}

__device__ __forceinline__ double2 to_d(double2 a) { return a; }
__device__ __forceinline__ double2 to_d(float2 a) { return to_c128(a); }
// The same for a matrix entry, converted where it is used: the plain
// conversion is loop-invariant and the compiler would keep the doubles.
__device__ __forceinline__ double2 entry_d(double2 a) { return a; }
__device__ __forceinline__ double2 entry_d(float2 a) {
  double2 d;
  asm volatile("v_cvt_f64_f32 %0, %1" : "=v"(d.x) : "v"(a.x));
  asm volatile("v_cvt_f64_f32 %0, %1" : "=v"(d.y) : "v"(a.y));
  return d;
}

// A thread's rows of Ahat = A D^-1: E entries per row, a row's missing ones
// zero in value and pointing at the row itself.  The values of the last EL
// entries of each row are in LDS (lv, [RPT][EL][NT]), where the registers do
// not take them all.
template <class V, int E, int EL, int RPT, int NT> struct ResRows {
  static constexpr int ER = E - EL;
  V a[RPT][ER];
  unsigned c[RPT][E];
  V* lv;

  // (row: the i-th of this thread where `has`; published at row + shift)
  template <class Args> __device__ __forceinline__ void load(int i, int row, bool has, int r0, int shift, const Args& A) {
    const int rc = has ? row : r0;
    const int s = A.rowptr[rc], len = has ? A.rowptr[rc + 1] - s : 0;
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int p = len > 0 ? s + min(k, len - 1) : 0;
      const int cc = A.col[p];
      const V q = A.scaled(p, cc);
      V v = k < len ? q : czero<V>();
      if (k % 4 == 3) here(v);
      if (k < ER) a[i][k] = v;
      else lv[(i * EL + k - ER) * NT + threadIdx.x] = v;
      c[i][k] = (unsigned)((k < len ? cc : rc) + shift) * (unsigned)sizeof(V);  // byte offset
    }
  }
  // Entry k ends a four; `part` and `acc` are the sums of its four and of the
  // row with av * xv added.
  static __device__ __forceinline__ constexpr bool ends(int k) { return (k - (E - 1) / 2) % 4 == 0 || k == E - 1; }
  static __device__ __forceinline__ void sum(int k, double2 av, double2 xv, double2& part, double2& acc) {
    part = k == 0 || ends(k - 1) ? cmul(av, xv) : cfma(av, xv, part);
    if (ends(k)) acc = k <= (E - 1) / 2 % 4 ? part : cadd(acc, part);
  }
  // Sum over the row's entries of a_k comb(k, ld(k, column)), the loads of
  // kGroup entries at a time issued ahead of the previous group's arithmetic:
  // left alone the compiler issues every load of the row at once and spills
  // the matrix.  The entries are summed four at a time, and a mesh row's middle
  // one, its diagonal, ends its four (`sum`): the largest partial sums are then
  // rounded every fourth entry.  One chain of multiply-adds over the row rounds
  // them twice per entry; its error on a random vector was 2.7e-16 of 15 entries
  // and 3.5e-16 of 27 against 1.5e-16 and 1.7e-16 with fours and 1.5e-16 to
  // 2.1e-16 and 1.7e-16 to 2.5e-16 in the row-block products (16 to 64 rows per
  // wave), and a BiCGStab(8) solve's true residual fell as much.  complex64
  // rows are summed in double: with a float chain the refinement cycles of the
  // mixed solve took up to twice the iterations of the kernels that sum a row's
  // products over lanes (279,496 rows, second cycle: 606 against 400-425 on
  // average), and the double one costs the same time, which the gathers set.
  template <class L, class C> __device__ __forceinline__ V dot(int i, L&& ld, C&& comb) const {
    constexpr int kBytes = E * RPT * (int)sizeof(V);
    constexpr int kGroup = kBytes <= 240 ? 4 : kBytes <= 440 ? 3 : 2, NG = (E + kGroup - 1) / kGroup;
    using X = decltype(ld(0, 0u));
    double2 acc = make_double2(0, 0), part = make_double2(0, 0);
    X x[2][kGroup];
#pragma unroll
    for (int k = 0; k < kGroup; ++k)
      if (k < E) x[0][k] = ld(k, fresh(c[i][k]));
#pragma unroll
    for (int g = 0; g < NG; ++g) {
#pragma unroll
      for (int k = 0; k < kGroup; ++k) {
        const int kk = (g + 1) * kGroup + k;
        if (kk < E) x[(g + 1) & 1][k] = ld(kk, fresh(c[i][kk]));
      }
#pragma unroll
      for (int k = 0; k < kGroup; ++k) {
        const int kk = g * kGroup + k;
        if (kk < ER) sum(kk, entry_d(a[i][kk]), to_d(comb(kk, x[g & 1][k])), part, acc);
        else if (kk < E) sum(kk, to_d(lv[(i * EL + kk - ER) * NT + threadIdx.x]), to_d(comb(kk, x[g & 1][k])), part, acc);
      }
      here(acc);
      if (!ends(min((g + 1) * kGroup, E) - 1)) here(part);
    }
    return vscal<V>(acc);
  }
};

template <int NT> struct ResLds {
  double sums[kSumWords * (NT / kWave + 4)];
};

// This workgroup's number of the `size` that solve a system: in the sums, and
// (at) among the rows.  A packed launch has kXcds times as many, of which every
// kXcds-th works: workgroups go to the XCDs in turn, so these share one, and with
// it the L2 that they publish to (same_xcd makes sure).
struct ResPlace {
  int size, rank, at;
  bool idle;
  __device__ __forceinline__ explicit ResPlace(int packed) {
    idle = packed && blockIdx.x % kXcds != 0;
    size = packed ? gridDim.x / kXcds : gridDim.x;
    rank = packed ? blockIdx.x / kXcds : blockIdx.x;
    at = packed ? rank : xcd_block(blockIdx.x, gridDim.x);
  }
};

// The row this thread works on as its i-th, and whether there is one.
template <int RPT, int NT> struct ResMap {
  int r0, rend;
  int shift = 0;  // row r is element r + shift of the published vectors
  __device__ __forceinline__ ResMap(int n, int rows, int at) {
    r0 = at * rows;
    rend = min(r0 + rows, n);
  }
  __device__ __forceinline__ ResMap(int from, int to, int end, int sh) : r0(from), rend(min(to, end)), shift(sh) {}
  __device__ __forceinline__ int row(int i) const { return r0 + i * NT + (int)threadIdx.x; }
  __device__ __forceinline__ int pub(int i) const { return row(i) + shift; }
  __device__ __forceinline__ bool has(int i) const { return row(i) < rend; }
};

// The first statuses of both methods (bb = ||b||^2, rr = ||r0||^2).
__device__ __forceinline__ int res_first_status(double bb, double rr, double theta2, long long maxit) {
  if (!isfinite(bb) || !isfinite(rr)) return HK_NONFINITE;
  if (rr <= theta2) return HK_OK;
  return maxit <= 0 ? HK_NOT_CONVERGED : S_RUN;
}

__device__ __forceinline__ void res_publish_state(SolveState* st, int status, int bd, double rr, double bb,
                                                  long long iter, long long iters_done) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  st->status = status;
  st->bd = bd;
  st->rr = rr;
  st->bb = bb;
  st->iter = iter;
  st->iters_done = iters_done;
}

// ------------------------------------------------------------------ host side

// Enqueues the solve on s: barrier words, state, then the cooperative
// launch.  hipErrorInvalidConfiguration (or what the launch gave) if it
// cannot run here.
template <class R> hipError_t resident_launch(const ResShape& sh, int method, ResArgs<R> args, void* scratch,
                                              hipStream_t s);
// The same for BiCGStab(l): l = ell; r_q at vecs + 2 q stride and u_q one stride
// behind it (q = 1 .. ell), read by their row's thread alone.
struct ResLArgs {
  ResArgs<double> base;
  int ell;
  double2* vecs;
  unsigned long long* many;  // words of grid_sum_many, all kSumEmpty at launch
};
hipError_t resident_l_launch(const ResShape& sh, ResLArgs args, void* scratch, hipStream_t s);
// The systems of a block-diagonal matrix (complex128 BiCGStab): system s is rows
// [row0, row1), `size` workgroups of `rows` rows, published at row + shift.  The
// shifts keep systems, which publish at different times, off each other's
// cache lines: a line that another system's workgroup on the same L2 has read
// in between would hide the newer content.
struct ResBatchSystem {
  int row0, row1, size, rows, shift;
};
struct ResBatchEnd {
  int status, bd;
  double rr, bb, rr_true;
  long long iters;
};
struct ResBatchArgs {
  ResArgs<double> base;       // gs.words: kSumSets * kSumSetWords for each system
  const ResBatchSystem* sys;
  // workgroup l (in XCD order) has jobs job_ptr[l] .. job_ptr[l + 1]: system and rank in it
  const int *job_ptr, *job_sys, *job_rank;
  double2* X;
  ResBatchEnd* end;
  int* running;  // systems that all of their workgroups have come to, 0 at launch
};
// Rows per thread (1 or 2), rows per workgroup and the job lists for systems of
// the given rows; false if one does not fit.
struct ResBatchPlan {
  int entries = 0, rpt = 0, grid = 0;
  int64_t stride = 0;  // elements of a published vector
  std::vector<ResBatchSystem> sys;
  std::vector<int> job_ptr, job_sys, job_rank;
};
bool resident_batch_plan(const hk_csr_s* A, int nsys, const int64_t* row_off, ResBatchPlan* plan);
hipError_t resident_batch_launch(const ResBatchPlan& plan, ResBatchArgs args, hipStream_t s);

// The systems (K - kappa_j M) x_j = b_j of a sweep (complex128 BiCGStab, K and M
// real): `groups` runs of `size` workgroups of `rows` rows take the systems from
// a queue, order[0 .. nsys), until it is empty.
struct ResSweepSource : ResArgs<double> {
  const double *K, *M, *kd, *md;  // values and diagonals
  double2 kappa;
  int j;  // b and x: column j of n x 64
  static __device__ __forceinline__ double2 of(double k, double m, double2 kappa) {
    return make_double2(fma(-kappa.x, m, k), -kappa.y * m);
  }
  __device__ __forceinline__ double2 entry(int p) const { return of(K[p], M[p], kappa); }
  __device__ __forceinline__ double2 inv_diag(int row) const {
    return cdiv(make_double2(1, 0), of(kd[row], md[row], kappa));
  }
  __device__ __forceinline__ double2 scaled(int p, int c) const { return cmul(entry(p), inv_diag(c)); }
  __device__ __forceinline__ double2 rhs(int row) const { return b[(size_t)row * kSweepLanes + j]; }
};
struct ResSweepArgs {
  ResSweepSource src;          // gs.words: kSumSets * kSumSetWords for each group
  const double2* kap;
  const int* order;
  int* next;                   // the queue's front, `groups` at launch
  int nsys, size, slots;       // slots: systems a group works on at a time
  int span, groups;            // groups lie within `span` workgroups in XCD order
  long long area;              // elements of a published vector of one system
  double2* own;                // slots > 1: what the slots keep per row
  unsigned long long* wide;    // and the words of group_sum_wide, all kSumEmpty at launch
  double2* X;
  ResBatchEnd* end;
};
// The group of this workgroup and its rank there.
struct ResGroup {
  int group, rank;
  bool idle;
  __device__ __forceinline__ explicit ResGroup(const ResSweepArgs& B) {
    const int l = xcd_block(blockIdx.x, gridDim.x), per = B.span / B.size, i = l % B.span;
    group = l / B.span * per + i / B.size;
    rank = i % B.size;
    idle = i / B.size >= per || group >= B.groups;
  }
};
struct ResSweepPlan {
  int entries = 0, rpt = 0, rows = 0, size = 0, groups = 0, slots = 1, grid = 0, span = 0;
  int64_t area = 0;
  // elements of the published vectors and of the slots' own ones; barrier words
  size_t pub() const { return (size_t)area * groups * (slots > 1 ? (2 * kRing + 1) * slots : 3 * kRing); }
  size_t own() const { return slots > 1 ? (size_t)area * groups * 2 * slots : 0; }
  size_t words() const;
};
constexpr int kManySlots = 6;  // what registers and LDS take
// hk_resident_sweep.hip: the kernel for `slots` > 1, the words of a group's
// group_sum_wide
const void* resident_many_kernel(const ResSweepPlan& plan);
size_t resident_many_words(int slots);
bool resident_sweep_plan(int device, int64_t n, int64_t nnz, int max_row, int nsys, ResSweepPlan* plan);
hipError_t resident_sweep_launch(const ResSweepPlan& plan, ResSweepArgs args, hipStream_t s);

// The barrier words at the front of the scratch emptied, the launch itself:
// kern with sh's grid and the argument struct at kargs[0], whose GridSum is gs.
hipError_t resident_launch_kernel(const void* kern, const ResShape& sh, void** kargs, GridSum* gs, void* scratch,
                                  hipStream_t s);
// All of `count` barrier words empty, the kResFlags ints at abort (which may lie
// behind them) 0.
constexpr size_t kResFlags = 32;
hipError_t resident_reset(unsigned long long* words, size_t count, int* abort, hipStream_t s);
// The abort flag in the scratch (device address), and the words behind it.
int* resident_abort(void* scratch);
unsigned long long* resident_many(void* scratch);

}  // namespace hk
