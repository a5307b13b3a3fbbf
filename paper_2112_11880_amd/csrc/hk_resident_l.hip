// hk_resident_l.hip -- BiCGStab(l) in one cooperative launch that keeps the
// matrix in registers (gfx950); see hk_resident.hip for the scheme and
// hk_solver.hip for the method's steps and statuses.
//
// As separate kernels a BiCG step on 232,897 rows took 75 us: two products of
// 17.8, the passes over the r_i and u_i of 10.5 and 8.6, finalize launches of 4.7
// each.  Here it takes 34 us: two barriers of 4, two gathers of two vectors for
// two rows per thread of 6-7, the pass over the r_i and u_i.  With j the step,
//   u_j = r_j - beta u_j:      u_{j+1} = Ahat u_j gathers the last r and u products
//   r_j - alpha u_{j+1}:       r_{j+1} = Ahat r_j gathers the last r and the new u
// so the two newest products of each kind are published (pub[0..1], pub[2..3] in
// turn) and nothing else.  The stop test on ||r_0||^2 shares the barrier of
// rt^H r_{j+1}, or of the Gram sums.  The other r_i and u_i are read by their row's
// thread alone, from memory: they do not fit beside the matrix, and both of a
// step's updates of them (r_i -= alpha u_{i+1}, then u_i = r_i - beta u_i) are one
// pass, after beta is known.  The l(l+3) Gram sums take grid_sum_many; one wave
// of each workgroup solves the l x l system, lane 8 i + k holding its entry (i, k).
#include "hk_resident.hpp"

namespace hk {

constexpr int kLMax = 8;

// Component (i, j), 0 <= i <= j < ell, of the Gram matrix behind the ell of the
// right-hand side.
__device__ __forceinline__ int gram_index(int i, int j, int ell) { return ell + i * ell - i * (i - 1) / 2 + (j - i); }

__device__ __forceinline__ double2 shfl2(double2 v, int lane) {
  return make_double2(__shfl(v.x, lane), __shfl(v.y, lane));
}

// gamma of Z gamma = z (totals: z, then Z's upper triangle, complex) into
// g[0..ell), by Cholesky in one wave; false (in every lane) if Z is not positive
// definite.
__device__ __forceinline__ bool gram_solve(const double* totals, int ell, double2* g) {
  const int lane = threadIdx.x % kWave, i = lane >> 3, k = lane & 7;
  const bool in = i < ell && k < ell;
  double2 Z = make_double2(0, 0), w = make_double2(0, 0);
  double rl = 0;
  if (in) {
    const int m = gram_index(min(i, k), max(i, k), ell);
    Z = make_double2(totals[2 * m], i <= k ? totals[2 * m + 1] : -totals[2 * m + 1]);
  }
  if (i < ell) w = make_double2(totals[2 * i], totals[2 * i + 1]);
#pragma unroll 1
  for (int j = 0; j < ell; ++j) {
    const double d = __shfl(Z.x, 9 * j);
    if (!(d > 0.0)) return false;
    const double ljj = sqrt(d), rj = 1.0 / ljj;
    double2 Lij = shfl2(Z, 8 * i + j), Lkj = shfl2(Z, 8 * k + j), wj = shfl2(w, 8 * j);
    Lij = make_double2(Lij.x * rj, Lij.y * rj);
    Lkj = make_double2(Lkj.x * rj, Lkj.y * rj);
    wj = make_double2(wj.x * rj, wj.y * rj);
    if (i > j && k > j) Z = csub(Z, cmul(Lij, cconj(Lkj)));
    if (k == j && i > j) Z = Lij;
    if (i > j) w = csub(w, cmul(Lij, wj));
    if (i == j) {
      w = wj;
      rl = rj;
    }
  }
#pragma unroll 1
  for (int j = ell - 1; j >= 0; --j) {
    const double2 wj = shfl2(w, 8 * j), Lji = shfl2(Z, 8 * j + i);
    const double rj = __shfl(rl, 8 * j);
    const double2 gj = make_double2(wj.x * rj, wj.y * rj);
    if (i < j) w = csub(w, cmul(cconj(Lji), gj));
    if (lane == 0) g[j] = gj;
  }
  return true;
}

template <int E, int EL, int RPT, int NT>
__global__ __launch_bounds__(NT, kResWaves) void k_res_bicgstab_l(ResLArgs L) {
  using V = double2;
  constexpr int W = NT / kWave;
  __shared__ ResLds<NT> lds;
  __shared__ double s_many[kManySums * W], s_tot[kManySums];
  __shared__ V s_g[kLMax];
  __shared__ int s_ok;
  __shared__ V s_rt[RPT * NT], s_y[RPT * NT], s_lv[EL > 0 ? RPT * EL * NT : 1];
  const ResArgs<double>& A = L.base;
  // r_q and u_q of the private vectors; the published r and u number c.  u is
  // read for the last time before the next step's first barrier and r before its
  // second, so with four places the caches are dropped at every other second
  // barrier, and where a cycle ends
  auto priv_r = [&](int q) { return L.vecs + 2 * q * A.stride; };
  auto priv_u = [&](int q) { return L.vecs + (2 * q + 1) * A.stride; };
  // a scalar base and a 32-bit offset, formed anew: 64-bit addresses by q are kept
  // and spilled (315 -> 238 and 46 -> 3 registers spilled with two and one rows of 15
  // entries per thread, a cycle of 16 products 296 -> 274 us on 232,897 rows, 135 ->
  // 123 on 117,649)
  auto get_priv = [](const V* base, int row) { return at(base, fresh((unsigned)row * (unsigned)sizeof(V))); };
  auto put_priv = [](V* base, int row, V v) {
    *reinterpret_cast<V*>(reinterpret_cast<char*>(base) + fresh((unsigned)row * (unsigned)sizeof(V))) = v;
  };
  auto pub = [&](int i, unsigned c) { return A.pub + (kRing * i + (int)(c & (kRing - 1))) * A.stride; };
  if (*A.flag) return;
  const int ell = L.ell, lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
  const ResPlace at_place(A.packed);
  if (at_place.idle) return;
  const int size = at_place.size, rank = at_place.rank;
  const ResMap<RPT, NT> m(A.n, A.rows, at_place.at);
  GridSum gs = A.gs;
  gs.local = 0;
  ResRows<V, E, EL, RPT, NT> M;
  M.lv = s_lv;
  V r0[RPT], u0[RPT], u1[RPT], un[RPT], rn[RPT];
  unsigned epoch = 0, many_calls = 0;
  unsigned np = 0;  // number of the newest r and u
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
      publish(gs, pub(0, 0), m.pub(i), ri);
      publish(gs, pub(1, 0), m.pub(i), czero<V>());
    }
    r0[i] = ri;
    u0[i] = u1[i] = un[i] = rn[i] = czero<V>();
    s_rt[l] = ri;
    s_y[l] = yi;
    sum2[0] += nrm2d(bi);
    sum2[1] += nrm2d(ri);
  }
  if (group_sum<4, NT>(gs, size, rank, epoch, true, sum2, lds.sums)) return;
  if (NT == 256) gs.local = same_xcd(size, sum2[2], sum2[3]);
  const bool first = rank == 0 && threadIdx.x == 0;
  const double bb = uni(sum2[0]), theta2 = uni(A.tol * A.tol * bb);
  double rr = uni(sum2[1]);
  V rho = make_double2(1, 0), alpha = czero<V>(), omega = make_double2(1, 0), beta = czero<V>();
  int status = res_first_status(bb, rr, theta2, A.maxit), bd = HK_BD_NONE;
  long long k = 1, done = 0;
  auto note = [&](long long at_k) {
    if (first && A.history) A.history[at_k] = bb > 0 ? sqrt(rr / bb) : 0.0;
  };
  // rho0 = -omega rho at a cycle's start, then beta = alpha rho1 / rho0, rho = rho1
  auto cycle_start = [&](V rho1) {
    const V rho0 = cmul(make_double2(-1, 0), cmul(omega, rho));
    if (!cfinite(rho1)) {
      status = HK_NONFINITE;
      done = k - 1;
    } else if (rho1.x == 0 && rho1.y == 0) {
      status = HK_BREAKDOWN;
      bd = HK_BD_RHO;
      done = k - 1;
    } else {
      beta = uni(cdiv(cmul(alpha, rho1), rho0));
      rho = rho1;
    }
  };
  // the stop test on ||r_0||^2 after a BiCG step
  auto stop_r = [&]() {
    if (!isfinite(rr)) {
      status = HK_NONFINITE;
      done = k;
    } else if (rr <= theta2) {
      status = HK_OK;
      done = k;
      note(k);
    }
  };
  note(0);
  if (status == S_RUN) cycle_start(make_double2(rr, 0));
  while (status == S_RUN) {
    for (int j = 0; j < ell; ++j) {
      const V *const pr = pub(0, np), *const pu = pub(1, np);
      V *const pr2 = pub(0, np + 1), *const pu2 = pub(1, np + 1);
      // u_{j+1} = Ahat u_j, u_j = r_j - beta u_j; rt^H u_{j+1}
      double sg[2] = {0, 0};
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        u0[i] = cfnma(beta, u0[i], r0[i]);
        un[i] = M.dot(
            i, [&](int, unsigned c) { return Pair<V>{at(pr, c), at(pu, c)}; },
            [&](int, const Pair<V>& x) { return cfnma(beta, x.v, x.u); });
        if (m.has(i)) {
          publish(gs, pu2, m.pub(i), un[i]);
          dotc_acc(s_rt[i * NT + threadIdx.x], un[i], sg[0], sg[1]);
        }
      }
      if (group_sum<2, NT>(gs, size, rank, epoch, false, sg, lds.sums)) return;
      const V gam = uni(make_double2(sg[0], sg[1]));
      if (!cfinite(gam)) {
        status = HK_NONFINITE;
        done = k - 1;
        break;
      }
      if (gam.x == 0 && gam.y == 0) {
        status = HK_BREAKDOWN;
        bd = HK_BD_SIGMA;
        done = k - 1;
        break;
      }
      alpha = uni(cdiv(rho, gam));
      // r_0 -= alpha u_1, y += alpha u_0, ||r_0||^2; r_{j+1} = Ahat r_j, rt^H r_{j+1}
      double rs[3] = {0, 0, 0};
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const int l = i * NT + threadIdx.x;
        r0[i] = cfnma(alpha, j == 0 ? un[i] : u1[i], r0[i]);
        s_y[l] = cfma(alpha, u0[i], s_y[l]);
        rn[i] = M.dot(
            i, [&](int, unsigned c) { return Pair<V>{at(pr, c), at(static_cast<const V*>(pu2), c)}; },
            [&](int, const Pair<V>& x) { return cfnma(alpha, x.v, x.u); });
        if (m.has(i)) {
          if (j + 1 < ell) publish(gs, pr2, m.pub(i), rn[i]);
          rs[0] += nrm2d(r0[i]);
          dotc_acc(s_rt[l], rn[i], rs[1], rs[2]);
        }
      }
      if (j + 1 == ell) {
        sum2[0] = rs[0];
        break;
      }
      if (group_sum<3, NT>(gs, size, rank, epoch, ((np + 1) & 1) == 0, rs, lds.sums)) return;
      ++np;
      rr = uni(rs[0]);
      stop_r();
      if (status != S_RUN) break;
      const V rho1 = uni(make_double2(rs[1], rs[2]));
      if (!cfinite(rho1)) {
        status = HK_NONFINITE;
        done = k - 1;
        break;
      }
      if (rho1.x == 0 && rho1.y == 0) {
        status = HK_BREAKDOWN;
        bd = HK_BD_RHO;
        done = k - 1;
        break;
      }
      beta = uni(cdiv(cmul(alpha, rho1), rho));
      rho = rho1;
      // r_q -= alpha u_{q+1}, u_q = r_q - beta u_q for q = 1 .. j, then the newest
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        if (!m.has(i)) continue;
        const int row = m.row(i);
        for (int q0 = 1; q0 <= j; q0 += 4) {
          V rq[4], uq[5];
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int q = min(q0 + s, j);
            rq[s] = get_priv(priv_r(q), row);
            uq[s] = get_priv(priv_u(q), row);
          }
          uq[4] = get_priv(priv_u(min(q0 + 4, j)), row);  // used only where it is u_{q0+4}
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int q = q0 + s;
            if (q > j) break;
            const V rv = cfnma(alpha, q == j ? un[i] : uq[s + 1], rq[s]);
            const V uv = cfnma(beta, uq[s], rv);
            put_priv(priv_r(q), row, rv);
            put_priv(priv_u(q), row, uv);
            if (q == 1) u1[i] = uv;
          }
        }
        const V uv = cfnma(beta, un[i], rn[i]);
        put_priv(priv_r(j + 1), row, rn[i]);
        put_priv(priv_u(j + 1), row, uv);
        if (j == 0) u1[i] = uv;
      }
    }
    if (status != S_RUN) break;
    // the last step's r_q -= alpha u_{q+1}; products r_a^H r_b, a = 1 .. ell, b = 0, a .. ell
    V x[RPT][kLMax + 1];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int row = m.has(i) ? m.row(i) : 0;
      V uq[kLMax + 1];
      x[i][0] = r0[i];
#pragma unroll
      for (int q = 1; q <= kLMax; ++q) {
        x[i][q] = uq[q] = czero<V>();
        if (q < ell && m.has(i)) {
          x[i][q] = get_priv(priv_r(q), row);
          uq[q] = get_priv(priv_u(q), row);
        }
      }
#pragma unroll
      for (int q = 1; q <= kLMax; ++q) {
        if (q == ell) {
          uq[q] = un[i];
          x[i][q] = rn[i];
        }
      }
#pragma unroll
      for (int q = 1; q < kLMax; ++q)
        if (q < ell) x[i][q] = cfnma(alpha, uq[q + 1], x[i][q]);
    }
    const int nz = ell + ell * (ell + 1) / 2;
    auto put = [&](int c, double v) {
      v = wave_sum63(v);
      if (lane == kWave - 1) s_many[c * W + wv] = v;
    };
#pragma unroll
    for (int a = 1; a <= kLMax; ++a) {
      if (a > ell) continue;
#pragma unroll
      for (int b = a - 1; b <= kLMax; ++b) {  // b = a - 1 stands for r_0
        if (b > ell) continue;
        double re = 0, im = 0;
#pragma unroll
        for (int i = 0; i < RPT; ++i) dotc_acc(x[i][a], x[i][b == a - 1 ? 0 : b], re, im);
        const int c = b == a - 1 ? a - 1 : gram_index(a - 1, b - 1, ell);
        put(2 * c, re);
        put(2 * c + 1, im);
      }
    }
    put(2 * nz, sum2[0]);
    if (grid_sum_many<NT>(gs, size, rank, L.many, many_calls, 2 * nz + 1, s_many, s_tot)) return;
    rr = uni(s_tot[2 * nz]);
    stop_r();
    if (status != S_RUN) break;
    if (wv == 0) {
      const bool ok = gram_solve(s_tot, ell, s_g);
      if (lane == 0) s_ok = ok;
    }
    __syncthreads();
    if (!s_ok) {
      status = HK_BREAKDOWN;
      bd = HK_BD_TAU;
      done = k;
      break;
    }
    omega = uni(s_g[ell - 1]);
    if (!cfinite(omega)) {
      status = HK_NONFINITE;
      done = k;
      break;
    }
    // y += sum gamma_j r_{j-1}, r_0 -= sum gamma_j r_j, u_0 -= sum gamma_j u_j; ||r_0||^2, rt^H r_0
    double mr[3] = {0, 0, 0};
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int l = i * NT + threadIdx.x, row = m.has(i) ? m.row(i) : 0;
      V uq[kLMax + 1];
#pragma unroll
      for (int q = 1; q <= kLMax; ++q) {
        uq[q] = czero<V>();
        if (q < ell && m.has(i)) uq[q] = get_priv(priv_u(q), row);
        if (q == ell) uq[q] = un[i];
      }
      V y = s_y[l], r = r0[i], u = u0[i];
#pragma unroll
      for (int q = 1; q <= kLMax; ++q) {
        if (q > ell) continue;
        const V g = s_g[q - 1];
        y = cfma(g, x[i][q - 1], y);
        r = cfnma(g, x[i][q], r);
        u = cfnma(g, uq[q], u);
      }
      s_y[l] = y;
      r0[i] = r;
      u0[i] = u;
      if (m.has(i)) {
        publish(gs, pub(0, np + 2), m.pub(i), r);
        publish(gs, pub(1, np + 2), m.pub(i), u);
        mr[0] += nrm2d(r);
        dotc_acc(s_rt[l], r, mr[1], mr[2]);
      }
    }
    if (group_sum<3, NT>(gs, size, rank, epoch, true, mr, lds.sums)) return;
    np += 2;
    rr = uni(mr[0]);
    done = k;
    note(k);
    if (!isfinite(rr)) {
      status = HK_NONFINITE;
    } else if (rr <= theta2) {
      status = HK_OK;
    } else if (omega.x == 0 && omega.y == 0) {
      status = HK_BREAKDOWN;
      bd = HK_BD_OMEGA;
    } else if (k >= A.maxit) {
      status = HK_NOT_CONVERGED;
    } else {
      ++k;
      cycle_start(uni(make_double2(mr[1], mr[2])));
    }
  }
#pragma unroll
  for (int i = 0; i < RPT; ++i)
    if (m.has(i)) A.y[m.row(i)] = s_y[i * NT + threadIdx.x];
  res_publish_state(A.st, status, bd, rr, bb, k, done);
}

hipError_t resident_l_launch(const ResShape& sh, ResLArgs args, void* scratch, hipStream_t s) {
  const void* kern = nullptr;
#define HK_RES(EE, EL, PP, TT) \
  if (sh.entries == EE && sh.rpt == PP && sh.threads == TT) kern = (const void*)k_res_bicgstab_l<EE, EL, PP, TT>;
  HK_RES(8, 0, 1, 256) HK_RES(8, 0, 1, 512) HK_RES(8, 2, 2, 512)
  HK_RES(15, 3, 1, 256) HK_RES(15, 3, 1, 512) HK_RES(15, 6, 2, 512)
  HK_RES(27, 13, 1, 256) HK_RES(27, 13, 1, 512)
#undef HK_RES
  args.base.rows = sh.rows;
  args.base.packed = sh.packed;
  args.many = resident_many(scratch);
  void* kargs[] = {&args};
  return resident_launch_kernel(kern, sh, kargs, &args.base.gs, scratch, s);
}

}  // namespace hk
