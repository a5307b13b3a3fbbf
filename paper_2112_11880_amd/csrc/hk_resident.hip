// hk_resident.hip -- Jacobi BiCGStab and TFQMR in one cooperative launch that
// keeps the matrix in registers (gfx950).
//
// A system of up to a few hundred thousand rows fits the register files of
// the chip: 256 CUs hold 128 MB of them, and the 27 MB of complex128 values of
// a 48^3 mesh (117,649 rows) take 75 registers of each of 117,649 threads, one
// row per thread.  Launched as separate kernels (hk_solver.hip) an iteration
// of such a system is bound by its eight launches and by the chains of
// dependent loads in each -- 28 us on 4,913 rows, 46-52 us on 117,649, where
// its bytes alone would take 0.3 and 9 us.  Here an iteration is three (TFQMR:
// two) barriers that also sum, group_sum in hk_grid.hpp, and between them
// row-local arithmetic and the products' gathers: 7 us on 4,913 rows (one XCD), 13.3 on
// 117,649 (3 us per barrier, 2-3 per gather of two vectors, which bound it now),
// TFQMR on 70,224 rows of 27 entries 66 -> 14.6 us, complex64 BiCGStab on 279,496
// rows 60 -> 21.8 us.
//
// What keeps the barriers so few: a product's operand is a combination, known
// only after the barrier's scalars, of vectors known before it, and every
// thread forms it where it gathers.
//   BiCGStab  p = r + beta q, q = p - omega v:  v = Ahat p gathers r and q
//             s = r - alpha v:                  t = Ahat s gathers r and v
//   TFQMR     y2 = y1 - alpha v:                u2 = Ahat y2 gathers y1 and v
//             y1' = w + beta y2:                u1 = Ahat y1' gathers w and y2
// The gathered combination is formed by the same operations as the owner's
// copy, so it has the same bits.  The vectors that are gathered are stored by
// their owners at agent scope (publish); everything else stays in the
// thread.  TFQMR's first half-step needs its scalars only for row-local
// updates, so both half-steps share one reduction.
//
// Row r of workgroup b: consecutive rows, one per lane, so that the gathers of
// entry k by a wave touch near-consecutive elements on a mesh in node order;
// xcd_block gives each XCD one range of the rows, whose vectors its L2 holds.
#include <cmath>
#include <utility>

#include "hk_resident.hpp"

namespace hk {

// How a solve ended.
struct ResEnd {
  int status, bd;
  double rr, bb;
  long long iter, iters_done;
};

// LDS of one BiCGStab solve.
template <class R, int EL, int RPT, int NT> struct ResBiLds {
  ResLds<NT> sums;
  cplx<R> rh[RPT * NT], y[RPT * NT], lv[EL > 0 ? RPT * EL * NT : 1];
};

// BiCGStab on the rows [r0, rend) of this workgroup, number `rank` of the `size`
// that solve the system: D x is left in lds.y.  LOC: they may find that they
// share an XCD.  `running`, if any: the systems that all of their workgroups have
// come to; the others of this one may still be at another.  Returns true if the
// kernel must stop.
template <class R, int E, int EL, int RPT, int NT, bool LOC, class Src>
__device__ __forceinline__ bool res_bicgstab(const Src& A, GridSum& gs, int size, int rank, unsigned& epoch,
                                             const ResMap<RPT, NT>& m, ResBiLds<R, EL, RPT, NT>& lds, ResEnd& end,
                                             int* running = nullptr) {
  using V = cplx<R>;
  // the rows' gathered r, kept from the v product for the t product where
  // the registers allow (15 fewer 16-byte gathers per row)
  constexpr bool kKeep = E * RPT * (int)sizeof(V) <= 256;
  V *const s_rh = lds.rh, *const s_y = lds.y;
  ResRows<V, E, EL, RPT, NT> M;
  M.lv = lds.lv;
  V r[RPT], q[RPT], p[RPT], v[RPT], t[RPT];
  // r, q and v of iteration `it` (r and q those it starts from).  All three are
  // read for the last time before the iteration's second barrier, so of the
  // third barriers of any kRing iterations in a row one drops the caches.
  auto pub = [&](int i, long long at_it) { return A.pub + (kRing * i + (int)(at_it & (kRing - 1))) * A.stride; };
  double sum2[4] = {0, 0, 0, 0};
  same_xcd_sums(sum2[2], sum2[3]);
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int row = m.row(i), l = i * NT + threadIdx.x;
    const bool has = m.has(i);
    M.load(i, row, has, m.r0, m.shift, A);
    V bi = czero<V>(), ri = czero<V>(), yi = czero<V>();
    if (has) {
      bi = A.rhs(row);
      ri = A.x0 ? A.r0[row] : bi;
      if (A.x0) yi = cdiv(A.x0[row], A.inv_diag(row));
      publish(gs, pub(0, 1), m.pub(i), ri);
      publish(gs, pub(1, 1), m.pub(i), czero<V>());
    }
    r[i] = ri;
    q[i] = p[i] = v[i] = t[i] = czero<V>();
    s_rh[l] = ri;
    s_y[l] = yi;
    sum2[0] += nrm2d(bi);
    sum2[1] += nrm2d(ri);
  }
  if (group_sum<4, NT>(gs, size, rank, epoch, true, sum2, lds.sums.sums, running)) return true;
  if (LOC) gs.local = same_xcd(size, sum2[2], sum2[3]);
  const bool first = rank == 0 && threadIdx.x == 0;
  if (running && first) atomicAdd(running, 1);
  const double bb = uni(sum2[0]), theta2 = uni(A.tol * A.tol * bb);
  double rr = uni(sum2[1]);
  double2 rho = make_double2(rr, 0), beta = make_double2(0, 0), alpha, omega;
  int status = res_first_status(bb, rr, theta2, A.maxit), bd = HK_BD_NONE;
  long long it = 1, done = 0;
  if (first && A.history) A.history[0] = bb > 0 ? sqrt(rr / bb) : 0.0;
  while (status == S_RUN) {
    const V *const pr = pub(0, it), *const pq = pub(1, it);
    V* const pv = pub(2, it);
    V rg[RPT][kKeep ? E : 1];
    // v = Ahat p, p = r + beta q; sigma = rhat^H v
    double sg[2] = {0, 0};
    {
      const V be = vscal<V>(beta);
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        p[i] = cfma(be, q[i], r[i]);
        v[i] = M.dot(
            i, [&](int, unsigned c) { return Pair<V>{at(pr, c), at(pq, c)}; },
            [&](int k, const Pair<V>& x) {
              if constexpr (kKeep) rg[i][k] = x.u;
              return cfma(be, x.v, x.u);
            });
        if (m.has(i)) {
          publish(gs, pv, m.pub(i), v[i]);
          dotc_acc(s_rh[i * NT + threadIdx.x], v[i], sg[0], sg[1]);
        }
      }
    }
    if (group_sum<2, NT>(gs, size, rank, epoch, false, sg, lds.sums.sums)) return true;
    const double2 sigma = make_double2(sg[0], sg[1]);
    if (!cfinite(sigma)) {
      status = HK_NONFINITE;
      done = it - 1;
      break;
    }
    if (sigma.x == 0 && sigma.y == 0) {
      status = HK_BREAKDOWN;
      bd = HK_BD_SIGMA;
      done = it - 1;
      break;
    }
    alpha = uni(cdiv(rho, sigma));
    const V al = vscal<V>(alpha);
    // t = Ahat s, s = r - alpha v; tau = t^H t, t^H s, ||s||^2
    double ts[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const V s = cfnma(al, v[i], r[i]);
      if constexpr (kKeep)
        t[i] = M.dot(
            i, [&](int, unsigned c) { return at<V>(pv, c); },
            [&](int k, V x) { return cfnma(al, x, rg[i][k]); });
      else
        t[i] = M.dot(
            i, [&](int, unsigned c) { return Pair<V>{at(pr, c), at<V>(pv, c)}; },
            [&](int, const Pair<V>& x) { return cfnma(al, x.v, x.u); });
      if (m.has(i)) {
        ts[0] += nrm2d(t[i]);
        dotc_acc(t[i], s, ts[1], ts[2]);
        ts[3] += nrm2d(s);
      }
    }
    if (group_sum<4, NT>(gs, size, rank, epoch, false, ts, lds.sums.sums)) return true;
    const double ss = ts[3];
    const bool half = isfinite(ss) && ss <= theta2;
    if (!half && (!isfinite(ss) || !isfinite(ts[0]) || !isfinite(ts[1]) || !isfinite(ts[2]))) {
      status = HK_NONFINITE;
      done = it - 1;
      break;
    }
    if (half || ts[0] == 0) {
      // converged on s, or tau = 0: y += alpha p
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const int l = i * NT + threadIdx.x;
        s_y[l] = cfma(al, p[i], s_y[l]);
      }
      rr = ss;
      done = it;
      status = half ? HK_OK : HK_BREAKDOWN;
      if (!half) bd = HK_BD_TAU;
      if (half && first && A.history) A.history[it] = bb > 0 ? sqrt(ss / bb) : 0.0;
      break;
    }
    omega = uni(make_double2(ts[1] / ts[0], ts[2] / ts[0]));
    const V om = vscal<V>(omega);
    // y += alpha p + omega s, r = s - omega t, q = p - omega v
    double xr[3] = {0, 0, 0};
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int l = i * NT + threadIdx.x;
      const V s = cfnma(al, v[i], r[i]);
      s_y[l] = cfma(om, s, cfma(al, p[i], s_y[l]));
      r[i] = cfnma(om, t[i], s);
      q[i] = cfnma(om, v[i], p[i]);
      if (m.has(i)) {
        publish(gs, pub(0, it + 1), m.pub(i), r[i]);
        publish(gs, pub(1, it + 1), m.pub(i), q[i]);
        xr[0] += nrm2d(r[i]);
        dotc_acc(s_rh[l], r[i], xr[1], xr[2]);
      }
    }
    if (group_sum<3, NT>(gs, size, rank, epoch, ((it + 1) & (kRing - 1)) == 0, xr, lds.sums.sums)) return true;
    rr = uni(xr[0]);
    done = it;
    const double2 rho1 = uni(make_double2(xr[1], xr[2]));
    if (first && A.history) A.history[it] = bb > 0 ? sqrt(rr / bb) : 0.0;
    if (!isfinite(rr) || !cfinite(rho1)) {
      status = HK_NONFINITE;
    } else if (rr <= theta2) {
      status = HK_OK;
    } else if (omega.x == 0 && omega.y == 0) {
      status = HK_BREAKDOWN;
      bd = HK_BD_OMEGA;
    } else if (rho1.x == 0 && rho1.y == 0) {
      status = HK_BREAKDOWN;
      bd = HK_BD_RHO;
    } else if (it >= A.maxit) {
      status = HK_NOT_CONVERGED;
    } else {
      beta = uni(cmul(cdiv(rho1, rho), cdiv(alpha, omega)));
      rho = rho1;
      ++it;
    }
  }
  end = ResEnd{status, bd, rr, bb, it, done};
  return false;
}

template <class R, int E, int EL, int RPT, int NT>
__global__ __launch_bounds__(NT, kResWaves) void k_res_bicgstab(ResArgs<R> A) {
  __shared__ ResBiLds<R, EL, RPT, NT> lds;
  if (*A.flag) return;
  const ResPlace at(A.packed);
  if (at.idle) return;
  const ResMap<RPT, NT> m(A.n, A.rows, at.at);
  GridSum gs = A.gs;
  gs.local = 0;
  ResEnd e;
  unsigned epoch = 0;
  if (res_bicgstab<R, E, EL, RPT, NT, NT == 256>(A, gs, at.size, at.rank, epoch, m, lds, e)) return;
#pragma unroll
  for (int i = 0; i < RPT; ++i)
    if (m.has(i)) A.y[m.row(i)] = lds.y[i * NT + threadIdx.x];
  res_publish_state(A.st, e.status, e.bd, e.rr, e.bb, e.iter, e.iters_done);
}

// What follows the solve of one of several systems: x = D^-1 y, published and
// stored by put(row, x), and the true residual ||b - A x||, whose place is end.
// Returns true if the kernel must stop.
template <int RPT, int NT, class Src, class Lds, class Put>
__device__ __forceinline__ bool res_finish(const Src& A, const GridSum& gs, int size, int rank, unsigned& epoch,
                                           const ResMap<RPT, NT>& m, Lds& lds, const ResEnd& e, ResBatchEnd* end,
                                           Put&& put) {
  using V = double2;
  V* const px = A.pub;  // r's first place: all of its readers are done
  double rt[1] = {0};
  __syncthreads();
  if (group_sum<1, NT>(gs, size, rank, epoch, true, rt, lds.sums.sums)) return true;
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    if (!m.has(i)) continue;
    const V x = cmul(A.inv_diag(m.row(i)), lds.y[i * NT + threadIdx.x]);
    put(m.row(i), x);
    publish(gs, px, m.pub(i), x);
  }
  if (group_sum<1, NT>(gs, size, rank, epoch, true, rt, lds.sums.sums)) return true;
  rt[0] = 0;
#pragma unroll 1
  for (int i = 0; i < RPT; ++i) {
    if (!m.has(i)) continue;
    const int row = m.row(i), p1 = A.rowptr[row + 1];
    V r = A.rhs(row);
    for (int p = A.rowptr[row]; p < p1; ++p) r = cfnma(A.entry(p), px[A.col[p] + m.shift], r);
    rt[0] += nrm2d(r);
  }
  if (group_sum<1, NT>(gs, size, rank, epoch, false, rt, lds.sums.sums)) return true;
  if (rank == 0 && threadIdx.x == 0) *end = ResBatchEnd{e.status, e.bd, e.rr, e.bb, rt[0], e.iters_done};
  return false;
}

// Systems of a block-diagonal matrix, each solved by as many workgroups as its
// rows need.  A workgroup works through the list of its systems (jobs), whose
// order is one order over all systems: the first unfinished one finds all its
// workgroups done with what comes before it, so every wait ends.  A workgroup that
// comes to a system early waits in its first barrier for whole solves of others,
// as long as these take: the limit of that wait counts only while no system runs,
// and one that runs has the limit at each of its own barriers.
template <int E, int EL, int RPT, int NT>
__global__ __launch_bounds__(NT) void k_res_batch(ResBatchArgs B) {
  __shared__ ResBiLds<double, EL, RPT, NT> lds;
  const ResArgs<double>& A = B.base;
  const int l = xcd_block(blockIdx.x, gridDim.x);
  for (int j = B.job_ptr[l]; j < B.job_ptr[l + 1]; ++j) {
    const int sys = __builtin_amdgcn_readfirstlane(B.job_sys[j]), rank = __builtin_amdgcn_readfirstlane(B.job_rank[j]);
    const ResBatchSystem S = B.sys[sys];
    GridSum gs = A.gs;
    gs.words += (size_t)sys * kSumSets * kSumSetWords;
    const ResMap<RPT, NT> m(S.row0 + rank * S.rows, S.row0 + rank * S.rows + S.rows, S.row1, S.shift);
    ResEnd e;
    unsigned epoch = 0;
    __syncthreads();
    if (res_bicgstab<double, E, EL, RPT, NT, true>(A, gs, S.size, rank, epoch, m, lds, e, B.running)) return;
    if (res_finish<RPT, NT>(A, gs, S.size, rank, epoch, m, lds, e, B.end + sys, [&](int row, double2 x) { B.X[row] = x; }))
      return;
    if (rank == 0 && threadIdx.x == 0) atomicAdd(B.running, -1);
  }
}

// The systems of a sweep, whose matrices K - kappa_j M are formed where the rows
// are loaded.  Each group of workgroups solves one system at a time and takes
// the next one from the queue: its first workgroup draws the number, a sum over
// the group hands it to the others.  The bits of a system's solution do not
// depend on the group.  A group's published vectors have places of their own, in
// whole cache lines, which its next system uses again: between the last reads
// of one system (before the sum that ends res_finish) and the first of the next
// lies the first barrier of its solve, which drops the caches.
// The interleaved launch (k_sweep) streams 20 vectors of all systems through HBM
// per iteration and meets at five barriers: 87 us per iteration for 32 systems of
// 4,913 rows and for 3, 173 for 4 of 110,160, 553 for 64 of 117,649.  Here one
// system's iteration takes 10 to 20 us and several run at a time: 14.9 -> 2.9 ms
// and 13.6 -> 2.0 ms the call, 86.9 -> 19.6, 304 -> 291.
template <int E, int EL, int RPT, int NT>
__global__ __launch_bounds__(NT) void k_res_sweep(ResSweepArgs B) {
  __shared__ ResBiLds<double, EL, RPT, NT> lds;
  ResSweepSource A = B.src;
  const ResGroup at(B);
  if (at.idle) return;
  const int group = at.group, rank = at.rank;
  const ResMap<RPT, NT> m(rank * A.rows, rank * A.rows + A.rows, A.n, (int)(group * B.area));
  GridSum gs = A.gs;
  gs.words += (size_t)group * kSumSets * kSumSetWords;
  unsigned epoch = 0;
  for (int q = group; q < B.nsys;) {
    const int sys = __builtin_amdgcn_readfirstlane(B.order[q]);
    A.j = sys;
    A.kappa = uni(B.kap[sys]);
    ResEnd e;
    __syncthreads();
    if (res_bicgstab<double, E, EL, RPT, NT, true>(A, gs, B.size, rank, epoch, m, lds, e)) return;
    if (res_finish<RPT, NT>(A, gs, B.size, rank, epoch, m, lds, e, B.end + sys,
                            [&](int row, double2 x) { B.X[(size_t)row * kSweepLanes + sys] = x; }))
      return;
    double next[1] = {0};
    if (rank == 0 && threadIdx.x == 0) next[0] = (double)atomicAdd(B.next, 1);
    __syncthreads();
    if (group_sum<1, NT>(gs, B.size, rank, epoch, false, next, lds.sums.sums)) return;
    q = __builtin_amdgcn_readfirstlane((int)next[0]);
  }
}


// TFQMR (complex128).  Statuses, counts and updates at each exit are those of
// the kernels in hk_solver.hip.
template <int E, int EL, int RPT, int NT>
__global__ __launch_bounds__(NT, kResWaves) void k_res_tfqmr(ResArgs<double> A) {
  using V = double2;
  __shared__ ResLds<NT> lds;
  __shared__ V s_rh[RPT * NT], s_y[RPT * NT], s_d[RPT * NT], s_lv[EL > 0 ? RPT * EL * NT : 1];
  if (*A.flag) return;
  const ResPlace at_place(A.packed);
  if (at_place.idle) return;
  const int size = at_place.size, rank = at_place.rank;
  const ResMap<RPT, NT> m(A.n, A.rows, at_place.at);
  GridSum gs = A.gs;
  gs.local = 0;
  ResRows<V, E, EL, RPT, NT> M;
  M.lv = s_lv;
  V y1[RPT], v[RPT], u1[RPT], w[RPT], y2[RPT], u2[RPT];
  // y1 and v that iteration k starts from, read for the last time before its
  // first barrier, and w and y2 of its half-steps, before its second: the caches
  // are dropped at one in kRing of each, y1 and v by second and w and y2 by first
  // barriers
  auto pub = [&](int i, long long at_k) { return A.pub + (kRing * i + (int)(at_k & (kRing - 1))) * A.stride; };
  unsigned epoch = 0;
  double sum2[4] = {0, 0, 0, 0};
  same_xcd_sums(sum2[2], sum2[3]);
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int row = m.row(i), l = i * NT + threadIdx.x;
    const bool has = m.has(i);
    M.load(i, row, has, m.r0, m.shift, A);
    V bi = czero<V>(), ri = czero<V>(), yi = czero<V>();
    if (has) {
      bi = A.b[row];
      ri = A.x0 ? A.r0[row] : bi;
      if (A.x0) yi = cdiv(A.x0[row], A.dinv[row]);
      publish(gs, pub(0, 1), m.pub(i), ri);
    }
    y1[i] = w[i] = ri;
    v[i] = u1[i] = y2[i] = u2[i] = czero<V>();
    s_rh[l] = ri;
    s_y[l] = yi;
    s_d[l] = czero<V>();
    sum2[0] += nrm2d(bi);
    sum2[1] += nrm2d(ri);
  }
  if (group_sum<4, NT>(gs, size, rank, epoch, true, sum2, lds.sums)) return;
  if (NT == 256) gs.local = same_xcd(size, sum2[2], sum2[3]);
  const bool first = rank == 0 && threadIdx.x == 0;
  const double bb = uni(sum2[0]), theta2 = uni(A.tol * A.tol * bb);
  double rr = uni(sum2[1]), tau = uni(sqrt(rr)), theta = 0;
  V rho = make_double2(rr, 0), alpha = czero<V>(), eta2 = czero<V>(), coef1 = czero<V>();
  int status = res_first_status(bb, rr, theta2, A.maxit), bd = HK_BD_NONE;
  long long k = 1, done = 0;
  if (first && A.history) A.history[0] = bb > 0 ? sqrt(rr / bb) : 0.0;
  // alpha and the d-update coefficient from sigma = rhat^H v; false at an exit
  auto sigma_step = [&](const double (&sg)[2]) {
    const V sigma = make_double2(sg[0], sg[1]);
    if (!cfinite(sigma)) {
      status = HK_NONFINITE;
      done = k - 1;
    } else if (sigma.x == 0 && sigma.y == 0) {
      status = HK_BREAKDOWN;
      bd = HK_BD_SIGMA;
      done = k - 1;
    } else {
      alpha = uni(cdiv(rho, sigma));
      coef1 = uni(cdiv(cmul(make_double2(theta * theta, 0), eta2), alpha));
    }
  };
  // theta, tau, eta and the bound of half-step h from ||w||^2; returns eta
  auto half_step = [&](double ww, long long h) {
    theta = uni(sqrt(ww) / tau);
    const double c = 1.0 / sqrt(1.0 + theta * theta);
    tau = uni(tau * theta * c);
    const V eta = uni(make_double2(c * c * alpha.x, c * c * alpha.y));
    const double bound = tau * sqrt((double)(h + 1));
    rr = uni(bound * bound);
    if (first && A.history) A.history[k] = bb > 0 ? bound / sqrt(bb) : 0.0;
    return eta;
  };
  if (status == S_RUN) {
    // v = u1 = Ahat y1
    double sg[2] = {0, 0};
    const V* const py1 = pub(0, 1);
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      u1[i] = M.dot(
          i, [&](int, unsigned c) { return at(py1, c); }, [&](int, V x) { return x; });
      v[i] = u1[i];
      if (m.has(i)) {
        publish(gs, pub(1, 1), m.pub(i), v[i]);
        dotc_acc(s_rh[i * NT + threadIdx.x], v[i], sg[0], sg[1]);
      }
    }
    if (group_sum<2, NT>(gs, size, rank, epoch, false, sg, lds.sums)) return;
    sigma_step(sg);
  }
  while (status == S_RUN) {
    const V *const py1 = pub(0, k), *const pv = pub(1, k);
    V *const pw = pub(2, k), *const py2 = pub(3, k);
    // half-steps 1 and 2: w -= alpha u1, ||w||^2; u2 = Ahat y2,
    // w -= alpha u2, ||w||^2, rhat^H w
    double hs[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      y2[i] = cfnma(alpha, v[i], y1[i]);
      w[i] = cfnma(alpha, u1[i], w[i]);
      const double w1 = nrm2d(w[i]);
      u2[i] = M.dot(
          i, [&](int, unsigned c) { return Pair<V>{at(py1, c), at(pv, c)}; },
          [&](int, const Pair<V>& x) { return cfnma(alpha, x.v, x.u); });
      w[i] = cfnma(alpha, u2[i], w[i]);
      if (m.has(i)) {
        publish(gs, pw, m.pub(i), w[i]);
        publish(gs, py2, m.pub(i), y2[i]);
        hs[0] += w1;
        hs[1] += nrm2d(w[i]);
        dotc_acc(s_rh[i * NT + threadIdx.x], w[i], hs[2], hs[3]);
      }
    }
    if (group_sum<4, NT>(gs, size, rank, epoch, (k & (kRing - 1)) == 0, hs, lds.sums)) return;
    const V eta1 = half_step(hs[0], 2 * k - 1);
    const V coef2 = uni(cdiv(cmul(make_double2(theta * theta, 0), eta1), alpha));
    done = k;
    if (!isfinite(tau) || !cfinite(eta1)) {
      status = HK_NONFINITE;
      break;
    }
    const bool half1 = rr <= theta2;
    V rho1 = czero<V>(), beta = czero<V>();
    if (half1) {
      status = HK_OK;
    } else {
      eta2 = half_step(hs[1], 2 * k);
      rho1 = uni(make_double2(hs[2], hs[3]));
      if (!isfinite(tau) || !cfinite(eta2)) status = HK_NONFINITE;
      else if (rr <= theta2) status = HK_OK;
      else if (!cfinite(rho1)) status = HK_NONFINITE;
      else if (rho1.x == 0 && rho1.y == 0) { status = HK_BREAKDOWN; bd = HK_BD_RHO; }
      else beta = uni(cdiv(rho1, rho));
    }
    // d = y1 + coef1 d, y += eta1 d; d = y2 + coef2 d, y += eta2 d
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int l = i * NT + threadIdx.x;
      const V d1 = cfma(coef1, s_d[l], y1[i]);
      V y = cfma(eta1, d1, s_y[l]);
      if (!half1) {
        const V d2 = cfma(coef2, d1, y2[i]);
        if (status != HK_NONFINITE) y = cfma(eta2, d2, y);
        s_d[l] = d2;
      }
      s_y[l] = y;
    }
    if (status != S_RUN) break;
    rho = rho1;
    if (k >= A.maxit) {
      status = HK_NOT_CONVERGED;
      break;
    }
    // y1 = w + beta y2; u1 = Ahat y1; v = u1 + beta (u2 + beta v)
    double sg[2] = {0, 0};
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      y1[i] = cfma(beta, y2[i], w[i]);
      u1[i] = M.dot(
          i, [&](int, unsigned c) { return Pair<V>{at<V>(py2, c), at<V>(pw, c)}; },
          [&](int, const Pair<V>& x) { return cfma(beta, x.u, x.v); });
      v[i] = cfma(beta, cfma(beta, v[i], u2[i]), u1[i]);
      if (m.has(i)) {
        publish(gs, pub(0, k + 1), m.pub(i), y1[i]);
        publish(gs, pub(1, k + 1), m.pub(i), v[i]);
        dotc_acc(s_rh[i * NT + threadIdx.x], v[i], sg[0], sg[1]);
      }
    }
    if (group_sum<2, NT>(gs, size, rank, epoch, ((k + 1) & (kRing - 1)) == 0, sg, lds.sums)) return;
    ++k;
    sigma_step(sg);
  }
#pragma unroll
  for (int i = 0; i < RPT; ++i)
    if (m.has(i)) A.y[m.row(i)] = s_y[i * NT + threadIdx.x];
  res_publish_state(A.st, status, bd, rr, bb, k, done);
}

// ------------------------------------------------------------------ host side

// Scratch: the words of group_sum, those of grid_sum_many, the flags.
constexpr size_t kResWords = kSumSets * kSumSetWords, kResMany = kManyWords;
__global__ void k_res_reset(unsigned long long* words, size_t count, int* abort) {
  const size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < count) words[i] = kSumEmpty;
  if (i < kResFlags) abort[i] = 0;
}
hipError_t resident_reset(unsigned long long* words, size_t count, int* abort, hipStream_t s) {
  hipLaunchKernelGGL(k_res_reset, dim3((unsigned)((count + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, words, count,
                     abort);
  return hipGetLastError();
}

size_t resident_scratch_bytes() { return sizeof(unsigned long long) * (kResWords + kResMany) + 256; }
int* resident_abort(void* scratch) {
  return reinterpret_cast<int*>(static_cast<unsigned long long*>(scratch) + kResWords + kResMany);
}
unsigned long long* resident_many(void* scratch) { return static_cast<unsigned long long*>(scratch) + kResWords; }

// Rows of up to 8, 15 (tetrahedra) or 27 (hexahedra) entries are held, up to
// kResMax rows per thread: what 256 registers of each of 512 threads and 160 KB
// of LDS per CU take.  Beyond it the values no longer fit.  Within it the
// resident launch is the faster one at every size (1.8M rows do not fit, 279,496
// in complex64 2.8x, 4,913 rows 4.5x with the recording of the graph that the
// separate kernels need), so there is no lower limit.
static int res_class(int max_row) { return max_row <= 8 ? 0 : max_row <= 15 ? 1 : 2; }
constexpr int kResEntries[3] = {8, 15, 27};
constexpr int kResMax[2][3] = {{2, 2, 1}, {4, 4, 2}};  // [complex64][class]

ResShape resident_shape(const hk_csr_s* A, int prec) {
  ResShape sh;
  if (A->plan_fixed || A->lean || A->nnz <= 0 || A->max_row > kResEntries[2]) return sh;
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, A->device) != hipSuccess) {
    (void)hipGetLastError();
    return sh;
  }
  cus = std::min(cus, kSumBlocks);
  const int cl = res_class(A->max_row), rpt_max = kResMax[prec][cl];
  int rpt = 1;
  while (rpt <= rpt_max && A->n > (int64_t)cus * 512 * rpt) ++rpt;
  if (rpt > rpt_max) return sh;
  // small systems: 256-thread workgroups, one wave per SIMD
  const int threads = A->n <= 64 * 256 ? 256 : 512;
  const int64_t even = rpt == 1 ? threads : (A->n + cus - 1) / cus;
  sh.rows = (int)((even + 63) / 64 * 64);
  sh.grid = (int)((A->n + sh.rows - 1) / sh.rows);
  sh.entries = kResEntries[cl];
  sh.rpt = rpt;
  sh.threads = threads;
  // on one XCD, two workgroups of 256 threads on each of its CUs at most: 4,913
  // rows (20 workgroups) 9.3 -> 7.1 us per iteration, set-up included
  sh.packed = threads == 256 && sh.grid <= 2 * (cus / kXcds) && sh.grid > 1;
  return sh;
}

// Time of one BiCGStab iteration in us, as measured: the barriers grow with the
// workgroups (9.6 us at 20, 13.3 at 230; on one XCD, whose groups share an L2, 7
// at 10 and 15 with two rows per thread at 30), a second row per thread costs the
// gathers again.
static double res_iteration_us(int size, int rpt, bool local) {
  return local ? 6.7 + 0.03 * size + 7.5 * (rpt - 1) : 9.3 + 0.0175 * size + 6.5 * (rpt - 1);
}
// Workgroups of a grid of G that share an XCD, consecutive in XCD order.
static int res_span(int G) { return G % kXcds == 0 ? G / kXcds : G; }

// Each system is given to the run of workgroups that is free first, the large
// ones first; with one or two rows per thread, whichever ends earlier (the
// iterations of a mesh's system taken as proportional to its rows' cube root).
bool resident_batch_plan(const hk_csr_s* A, int nsys, const int64_t* row_off, ResBatchPlan* plan) {
  if (A->nnz <= 0 || A->max_row > kResEntries[2]) return false;
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, A->device) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  const int G = std::min(cus, kSumBlocks), cl = res_class(A->max_row), span = res_span(G);
  std::vector<int> order(nsys);
  for (int k = 0; k < nsys; ++k) order[k] = k;
  auto rows_of = [&](int k) { return row_off[k + 1] - row_off[k]; };
  std::stable_sort(order.begin(), order.end(), [&](int p, int q) { return rows_of(p) > rows_of(q); });
  double best = -1;
  for (int rpt = 1; rpt <= kResMax[0][cl]; ++rpt) {
    if (rows_of(order[0]) > (int64_t)G * 512 * rpt) continue;
    ResBatchPlan p;
    p.entries = kResEntries[cl];
    p.rpt = rpt;
    p.grid = G;
    p.sys.resize(nsys);
    std::vector<double> free_at(G, 0.0);
    std::vector<std::vector<std::pair<int, int>>> jobs(G);
    double end = 0;
    for (int k = 0; k < nsys; ++k) {
      // 64 elements: whole cache lines
      p.sys[k].shift = (int)(p.stride - row_off[k]);
      p.stride += (rows_of(k) + 63) / 64 * 64;
    }
    for (int k : order) {
      ResBatchSystem& s = p.sys[k];
      s.row0 = (int)row_off[k];
      s.row1 = (int)row_off[k + 1];
      const int least = (int)((rows_of(k) + 512 * rpt - 1) / (512 * rpt));
      s.rows = (int)(((rows_of(k) + least - 1) / least + 63) / 64 * 64);
      s.size = (int)((rows_of(k) + s.rows - 1) / s.rows);
      int at = 0;
      double when = -1;
      // on one XCD where it fits
      const bool local = s.size <= span;
      for (int l = 0; l + s.size <= G; ++l) {
        if (local && l / span != (l + s.size - 1) / span) continue;
        double t = 0;
        for (int q = l; q < l + s.size; ++q) t = std::max(t, free_at[q]);
        if (when < 0 || t < when) { when = t; at = l; }
      }
      const double t = when + std::cbrt((double)rows_of(k)) * res_iteration_us(s.size, rpt, local);
      for (int q = 0; q < s.size; ++q) {
        free_at[at + q] = t;
        jobs[at + q].push_back({k, q});
      }
      end = std::max(end, t);
    }
    p.job_ptr.push_back(0);
    for (const auto& v : jobs) {
      for (const auto& jb : v) {
        p.job_sys.push_back(jb.first);
        p.job_rank.push_back(jb.second);
      }
      p.job_ptr.push_back((int)p.job_sys.size());
    }
    if (best < 0 || end < best) {
      best = end;
      *plan = std::move(p);
    }
  }
  return best >= 0;
}

// kern with `grid` workgroups of 512 threads, all of them resident.
template <class Args> static hipError_t res_coop_launch(const void* kern, int grid, Args& args, hipStream_t s) {
  if (!kern) return hipErrorInvalidConfiguration;
  int per = 0, cus = 0, coop = 0, dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, 512, 0);
  if (e != hipSuccess) return e;
  if (!coop || grid > per * cus) return hipErrorInvalidConfiguration;
  void* kargs[] = {&args};
  return hipLaunchCooperativeKernel(kern, dim3(grid), dim3(512), kargs, 0, s);
}

hipError_t resident_batch_launch(const ResBatchPlan& plan, ResBatchArgs args, hipStream_t s) {
  const void* kern = nullptr;
#define HK_RES(EE, EL, PP) \
  if (plan.entries == EE && plan.rpt == PP) kern = (const void*)k_res_batch<EE, EL, PP, 512>;
  HK_RES(8, 0, 1) HK_RES(8, 2, 2) HK_RES(15, 0, 1) HK_RES(15, 6, 2) HK_RES(27, 13, 1)
#undef HK_RES
  return res_coop_launch(kern, plan.grid, args, s);
}

// Time of one iteration of `slots` systems at a time in us, as measured: 26 and 43
// with 3 and 6 slots of 59 workgroups, 33 with 4 of 216, 31 and 45 with 3 and 6 of
// 230.
static double many_iteration_us(int size, int slots, bool local) {
  return (local ? 7 : 12) + 0.02 * size + 4.6 * slots;
}

size_t ResSweepPlan::words() const {
  return (size_t)groups * (kSumSets * kSumSetWords + (slots > 1 ? resident_many_words(slots) : 0));
}
// Rows per thread, or systems at a time: whichever gets through the systems in
// less time, taken in rounds of one system per group, or as long as the slots
// are full (each is filled again as soon as it is free).  64 systems of 117,649
// rows: 291 ms with two rows per thread (two groups of one system), 212 with six
// slots; two systems are faster with a group each (20 us per iteration against
// 29).
bool resident_sweep_plan(int device, int64_t n, int64_t nnz, int max_row, int nsys, ResSweepPlan* plan) {
  // a system of one workgroup stays with the interleaved launch, not for its
  // speed (63 iterations of 3 systems: 5.0 ms at 512 rows, 0.68 resident at 513)
  // but because that launch records the barrier times: at such sizes a call with
  // the record and one without give the same bits, as they always have
  if (n <= 512 || nnz <= 0 || max_row > kResEntries[2]) return false;
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  const int G = std::min(cus, kSumBlocks), cl = res_class(max_row), xcd = res_span(G);
  double best = -1;
  for (int rpt = 1; rpt <= kResMax[0][cl]; ++rpt) {
    const int64_t least = (n + 512 * rpt - 1) / (512 * rpt);
    if (least > G) continue;
    ResSweepPlan p;
    p.entries = kResEntries[cl];
    p.rpt = rpt;
    p.rows = (int)(((n + least - 1) / least + 63) / 64 * 64);
    p.size = (int)((n + p.rows - 1) / p.rows);
    p.area = (n + 63) / 64 * 64;  // whole cache lines
    // over the whole chip, and with every group on one XCD
    for (int span : {G, xcd}) {
      if (p.size > span || (span == G && p.size <= 1)) continue;
      const bool local = span == xcd && xcd < G;
      p.entries = kResEntries[cl];
      p.slots = 1;
      p.groups = std::min(G / span * (span / p.size), nsys);
      p.grid = local ? G : p.size * p.groups;
      p.span = local ? span : p.grid;
      auto take = [&](double us) {
        const int at_a_time = p.groups * p.slots;
        const double rounds = p.slots > 1 ? std::max(1.0, (double)nsys / at_a_time) : (nsys + at_a_time - 1) / at_a_time;
        const double t = rounds * us;
        if (best < 0 || t < best) {
          best = t;
          *plan = p;
        }
      };
      take(res_iteration_us(p.size, rpt, local));
      if (rpt == 1 && cl <= 1) {
        p.entries = 15;
        p.slots = std::min((nsys + p.groups - 1) / p.groups, kManySlots);
        if (p.slots > 1) take(many_iteration_us(p.size, p.slots, local));
      }
      if (xcd == G) break;
    }
  }
  return best >= 0;
}

hipError_t resident_sweep_launch(const ResSweepPlan& plan, ResSweepArgs args, hipStream_t s) {
  const void* kern = nullptr;
#define HK_RES(EE, EL, PP) \
  if (plan.entries == EE && plan.rpt == PP) kern = (const void*)k_res_sweep<EE, EL, PP, 512>;
  HK_RES(8, 0, 1) HK_RES(8, 2, 2) HK_RES(15, 0, 1) HK_RES(15, 6, 2) HK_RES(27, 13, 1)
#undef HK_RES
  if (plan.slots > 1) kern = resident_many_kernel(plan);
  args.src.rows = plan.rows;
  args.src.stride = plan.area * plan.groups;
  args.size = plan.size;
  args.slots = plan.slots;
  args.area = plan.area;
  args.wide = args.src.gs.words + (size_t)plan.groups * kSumSets * kSumSetWords;
  args.span = plan.span;
  args.groups = plan.groups;
  return res_coop_launch(kern, plan.grid, args, s);
}

template <class R> static const void* res_kernel(const ResShape& sh, int method) {
#define HK_RES(EE, EL, PP, TT)                                                        \
  if (sh.entries == EE && sh.rpt == PP && sh.threads == TT) {                         \
    if (method == HK_BICGSTAB) return (const void*)k_res_bicgstab<R, EE, EL, PP, TT>; \
    if constexpr (sizeof(R) == 8) return (const void*)k_res_tfqmr<EE, EL, PP, TT>;    \
  }
  if constexpr (sizeof(R) == 8) {
    HK_RES(8, 0, 1, 256) HK_RES(8, 0, 1, 512) HK_RES(8, 2, 2, 512)
    HK_RES(15, 0, 1, 256) HK_RES(15, 0, 1, 512) HK_RES(15, 6, 2, 512)
    HK_RES(27, 13, 1, 256) HK_RES(27, 13, 1, 512)
  } else {
    HK_RES(8, 0, 1, 256) HK_RES(8, 0, 1, 512) HK_RES(8, 0, 2, 512) HK_RES(8, 0, 3, 512) HK_RES(8, 2, 4, 512)
    HK_RES(15, 0, 1, 256) HK_RES(15, 0, 1, 512) HK_RES(15, 0, 2, 512) HK_RES(15, 4, 3, 512) HK_RES(15, 7, 4, 512)
    HK_RES(27, 0, 1, 256) HK_RES(27, 0, 1, 512) HK_RES(27, 12, 2, 512)
  }
#undef HK_RES
  return nullptr;
}

hipError_t resident_launch_kernel(const void* kern, const ResShape& sh, void** kargs, GridSum* gs, void* scratch,
                                  hipStream_t s) {
  if (!kern) return hipErrorInvalidConfiguration;
  int per = 0, cus = 0, coop = 0, dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, sh.threads, 0);
  if (e != hipSuccess) return e;
  const int grid = sh.packed ? sh.grid * kXcds : sh.grid;
  if (!coop || grid > per * cus || sh.grid > kSumBlocks || sh.rows > sh.rpt * sh.threads)
    return hipErrorInvalidConfiguration;
  gs->words = static_cast<unsigned long long*>(scratch);
  gs->abort = resident_abort(scratch);
  gs->spin_limit = barrier_spin_limit();
  e = resident_reset(gs->words, kResWords + kResMany, gs->abort, s);
  if (e != hipSuccess) return e;
  return hipLaunchCooperativeKernel(kern, dim3(grid), dim3(sh.threads), kargs, 0, s);
}

template <class R>
hipError_t resident_launch(const ResShape& sh, int method, ResArgs<R> args, void* scratch, hipStream_t s) {
  args.rows = sh.rows;
  args.packed = sh.packed;
  void* kargs[] = {&args};
  return resident_launch_kernel(res_kernel<R>(sh, method), sh, kargs, &args.gs, scratch, s);
}
template hipError_t resident_launch<double>(const ResShape&, int, ResArgs<double>, void*, hipStream_t);
template hipError_t resident_launch<float>(const ResShape&, int, ResArgs<float>, void*, hipStream_t);

}  // namespace hk
