// hk_resident_sweep.hip -- several systems of a sweep at a time on workgroups that
// keep K and M in registers (gfx950).
//
// k_res_sweep (hk_resident.hip) gives a group of workgroups one system, whose
// iteration is three barriers and gathers of four vectors.  On 117,649 rows two
// groups of 115 workgroups take 20 us for an iteration of each: the gathers
// (four vectors, 15 entries of 16 bytes for the 1,024 rows of a CU, 6.4 us at the
// 64 bytes per clock of its L1) and the barriers share the time.  The systems of
// a sweep have K and M in common, so here a thread has one row, K and M in
// registers once, and the state of up to G systems (slots) beside them:
//   r (s) and p in registers, v, t and D x in LDS, rhat and D^-1 in memory,
// and the barriers are met for all of them together.  As they cost each system
// 1/G, there are five: p and s are published scaled by D^-1 (two vectors to
// gather instead of four), in between the three that sum.  Systems that have
// ended are replaced from the queue between two iterations, at two more barriers:
// the slots that ended get their true residual, the next systems their ||b||.
//
// Six slots on 117,649 rows: 45 us, of which the five barriers 20, the two
// products 14 (1.2 us for each system's, 0.8 at the L1's rate), the updates 11
// (the published vectors' stores go past the L2: 11 MB each in 4 us).  64 systems
// 291 -> 212 ms, 20 of 110,160 rows 87 -> 66, 64 of 29,791 rows 42 -> 32.  What
// did not help: eight slots (what no longer fits goes to memory or is spilled, 65
// us), products in groups of four loads as elsewhere (the slots' products follow
// each other, each waits for its loads once instead of four times), slots in one
// unrolled loop with the product (180 KB of code: 123 us).
#include <cmath>
#include <type_traits>

#include "hk_resident.hpp"

namespace hk {

// What the workgroup knows of the systems in its slots, written by wave 0.
template <int G> struct MultiLds {
  double2 kap[G], rho[G], alpha[G], beta[G], omega[G];
  double bb[G], theta2[G], rr[G], ss[G];
  long long it[G], done[G];
  int sys[G], status[G], bd[G];
  unsigned run, half;  // slots that iterate; that end with y += alpha p
};

template <int E, int G, int NT, bool LOC>
__global__ __launch_bounds__(NT) void k_res_sweep_many(ResSweepArgs B) {
  using V = double2;
  constexpr int W = NT / kWave, NP = G <= 4 ? 8 : 16;  // up to four sums per slot
  __shared__ V s_v[G * NT], s_t[G * NT], s_y[G * NT];
  __shared__ MultiLds<G> L;
  __shared__ double s_waves[4 * G * W], s_parts[2 * NP * W], s_sums[kSumWords * (W + 4)];
  const ResSweepSource& A = B.src;
  const ResGroup place(B);
  if (place.idle) return;
  const int group = place.group, rank = place.rank;
  const ResMap<1, NT> m(rank * A.rows, rank * A.rows + A.rows, A.n, 0);
  const bool has = m.has(0);
  const int row = m.row(0), slots = B.slots;
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave, tid = threadIdx.x;
  GridSum gs = A.gs;
  gs.local = 0;
  gs.words += (size_t)group * kSumSets * kSumSetWords;
  unsigned long long* const wide = B.wide + (size_t)group * WideSum<NP>::kWords;
  unsigned epoch = 0, wepoch = 0;
  // published vectors of this group: vector i (p, s), place q, slot g, then x
  V* const pubs = A.pub + (size_t)group * (2 * kRing + 1) * slots * B.area;
  auto pub = [&](int i, unsigned q, int g) { return pubs + ((size_t)(kRing * i + (q & (kRing - 1))) * slots + g) * B.area; };
  const unsigned at_row = (unsigned)(has ? row : m.r0);
  // rows' own values in memory, by slot
  enum { RHAT, DINV };
  V* const owns = B.own + (size_t)group * 2 * slots * B.area;
  auto own_at = [&](int i, int g) { return owns + ((size_t)i * slots + g) * B.area; };
  auto own = [&](int i, int g) { return at(own_at(i, min(g, slots - 1)), fresh(at_row) * (unsigned)sizeof(V)); };
  auto put_own = [&](int i, int g, V v) {
    *reinterpret_cast<V*>(reinterpret_cast<char*>(own_at(i, g)) + fresh(at_row) * (unsigned)sizeof(V)) = v;
  };
  // row's entries
  double K[E], M[E];
  unsigned c[E];
  {
    const int rc = has ? row : m.r0;
    const int p0 = A.rowptr[rc], len = has ? A.rowptr[rc + 1] - p0 : 0;
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int p = len > 0 ? p0 + min(k, len - 1) : 0;
      K[k] = k < len ? A.K[p] : 0.0;
      M[k] = k < len ? A.M[p] : 0.0;
      c[k] = (unsigned)(k < len ? A.col[p] : rc) * (unsigned)sizeof(V);
    }
  }
  // (each slot's addresses anew: kept across the loop they take more registers than the slots)
  auto at_v = [&](int g) -> V& { return s_v[g * NT + fresh(threadIdx.x)]; };
  auto at_y = [&](int g) -> V& { return s_y[g * NT + fresh(threadIdx.x)]; };
  auto at_t = [&](int g) -> V& { return s_t[g * NT + fresh(threadIdx.x)]; };
  V r[G], p[G];
#pragma unroll
  for (int g = 0; g < G; ++g) r[g] = p[g] = czero<V>();
  // (K - kappa M) z of this row, z published at `base`
  auto product = [&](const V* base, V kap) {
    V ak = czero<V>(), am = czero<V>(), x[E];
#pragma unroll
    for (int k = 0; k < E; ++k) x[k] = at(base, fresh(c[k]));
#pragma unroll
    for (int k = 0; k < E; ++k) {
      ak.x = fma(K[k], x[k].x, ak.x);
      ak.y = fma(K[k], x[k].y, ak.y);
      am.x = fma(M[k], x[k].x, am.x);
      am.y = fma(M[k], x[k].y, am.y);
    }
    return cfnma(kap, am, ak);
  };
  // the wave's part of slot g's N sums (zeros behind them)
  auto put = [&](auto N, int g, const double (&v)[4]) {
    constexpr int n = decltype(N)::value;
    const double s = wave_sums4(v[0], v[1], v[2], v[3]);
    const int l4 = lane >> 4, i = l4 == 1 ? 2 : l4 == 2 ? 1 : l4;
    if ((lane & 15) == 15 && i < n) s_waves[(g * n + i) * W + w] = s;
  };
  constexpr std::integral_constant<int, 2> two{};
  constexpr std::integral_constant<int, 3> three{};
  constexpr std::integral_constant<int, 4> four{};
  // (wave 0, lane g) the total
  auto total = [&](int i, int n, int g) {
    double s = 0;
#pragma unroll
    for (int j = 0; j < W; ++j) s += s_parts[(g * n + i) * W + j];
    return s;
  };
  auto masks = [&](int g) {  // (wave 0)
    const int st = g < slots ? L.status[g] : HK_OK;
    const unsigned run = (unsigned)__ballot(st == S_RUN), half = (unsigned)__ballot(st == S_HALF || st == S_TAUBD);
    if (g == 0) { L.run = run; L.half = half; }
  };
  if (tid < G) {
    L.sys[tid] = -1;
    L.status[tid] = HK_OK;
    L.kap[tid] = czero<V>();
  }
  __syncthreads();
  unsigned occ = 0;      // slots that hold a system
  bool more = true;      // the queue may have one
  for (unsigned turn = 0;; ++turn) {
    // systems that ended, and those that take their place
    for (;;) {
      const unsigned run = turn == 0 && occ == 0 ? 0u : __builtin_amdgcn_readfirstlane(L.run);
      const unsigned fin = occ & ~run, all = slots >= 32 ? ~0u : (1u << slots) - 1;
      unsigned open = all & ~run;
      if (!fin && !(more && open)) break;
      if (!more) open = 0;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (!(fin >> g & 1)) continue;
        if (has) {
          const V x = cmul(own(DINV, g), at_y(g));
          B.X[(size_t)row * kSweepLanes + L.sys[g]] = x;
          publish(gs, pubs + ((size_t)2 * kRing * slots + g) * B.area, fresh(at_row), x);
        }
      }
      double from[3] = {0, 0, 0};
      same_xcd_sums(from[1], from[2]);
      if (rank == 0 && tid == 0 && open) from[0] = (double)atomicAdd(B.next, __popc(open));
      if (group_sum<3, NT>(gs, B.size, rank, epoch, true, from, s_sums)) return;
      if (LOC) gs.local = same_xcd(B.size, from[1], from[2]);
      int q = __builtin_amdgcn_readfirstlane((int)from[0]);
      unsigned fresh_ones = 0;
      // two sums per slot: the residual of its last system, ||b||^2 of its next
#pragma unroll 1
      for (int g = 0; g < slots; ++g) {
        if (!(fin >> g & 1)) continue;
        const V ax = product(pubs + ((size_t)2 * kRing * slots + g) * B.area, L.kap[g]);
        if (has) at_t(g).x = nrm2d(csub(own(RHAT, g), ax));
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (g >= slots) continue;
        double sums[4] = {0, 0, 0, 0};
        if (fin >> g & 1 && has) sums[0] = at_t(g).x;
        if (open >> g & 1) {
          if (q < B.nsys) {
            const int sys = __builtin_amdgcn_readfirstlane(B.order[q]);
            fresh_ones |= 1u << g;
            const V kap = B.kap[sys];
            V b = czero<V>();
            if (has) {
              b = A.b[(size_t)row * kSweepLanes + sys];
              put_own(RHAT, g, b);
              put_own(DINV, g, cdiv(make_double2(1, 0), A.of(A.kd[row], A.md[row], kap)));
            }
            r[g] = b;
            p[g] = czero<V>();
            at_v(g) = at_y(g) = czero<V>();
            sums[1] = nrm2d(b);
          } else {
            more = false;
          }
          ++q;
        }
        put(two, g, sums);
      }
      if (group_sum_wide<NP, NT>(gs, wide, B.size, rank, wepoch, 2 * slots, s_waves, s_parts)) return;
      if (w == 0) {
        const int g = lane;
        if (g < slots) {
          if (fin >> g & 1) {
            if (rank == 0)
              B.end[L.sys[g]] = ResBatchEnd{L.status[g], L.bd[g], L.rr[g], L.bb[g], total(0, 2, g), L.done[g]};
            L.sys[g] = -1;
            L.status[g] = HK_OK;
          }
          if (fresh_ones >> g & 1) {
            const double bb = total(1, 2, g);
            const int at_q = (int)from[0] + __popc(open & ((1u << g) - 1));
            const int sys = B.order[at_q];
            L.sys[g] = sys;
            L.kap[g] = B.kap[sys];
            L.bb[g] = L.rr[g] = bb;
            L.theta2[g] = A.tol * A.tol * bb;
            L.rho[g] = make_double2(bb, 0);
            L.beta[g] = L.omega[g] = czero<V>();
            L.it[g] = 1;
            L.done[g] = 0;
            L.bd[g] = HK_BD_NONE;
            L.status[g] = res_first_status(bb, bb, L.theta2[g], A.maxit);
          }
        }
        masks(lane);
      }
      __syncthreads();
      occ = (occ & ~fin) | fresh_ones;
    }
    if (!occ) return;
    // p = r + beta (p - omega v)
    unsigned run = __builtin_amdgcn_readfirstlane(L.run);
    V m1[G];
#pragma unroll
    for (int g = 0; g < G; ++g) m1[g] = own(DINV, g);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (!(run >> g & 1)) continue;
      p[g] = cfma(L.beta[g], cfnma(L.omega[g], at_v(g), p[g]), r[g]);
      if (has) publish(gs, pub(0, turn, g), fresh(at_row), cmul(m1[g], p[g]));
    }
    // both vectors' places were last read before the barriers of the turn before
    {
      double none[1] = {0};
      if (group_sum<1, NT>(gs, B.size, rank, epoch, (turn & (kRing - 1)) == 0, none, s_sums)) return;
    }
    // v = A D^-1 p; sigma = rhat^H v
#pragma unroll 1
    for (int g = 0; g < slots; ++g) {
      // (the sums of threads without a row are zero: their entries are)
      double sums[4] = {0, 0, 0, 0};
      if (run >> g & 1) {
        const V rh = own(RHAT, g), v = product(pub(0, turn, g), L.kap[g]);
        at_v(g) = v;
        dotc_acc(rh, v, sums[0], sums[1]);
      }
      put(two, g, sums);
    }
    if (group_sum_wide<NP, NT>(gs, wide, B.size, rank, wepoch, 2 * slots, s_waves, s_parts)) return;
    if (w == 0) {
      const int g = lane;
      if (run >> g & 1 && g < G) {
        const V sigma = make_double2(total(0, 2, g), total(1, 2, g));
        if (!cfinite(sigma)) {
          L.status[g] = HK_NONFINITE;
          L.done[g] = L.it[g] - 1;
        } else if (sigma.x == 0 && sigma.y == 0) {
          L.status[g] = HK_BREAKDOWN;
          L.bd[g] = HK_BD_SIGMA;
          L.done[g] = L.it[g] - 1;
        } else {
          L.alpha[g] = cdiv(L.rho[g], sigma);
        }
      }
      masks(lane);
    }
    __syncthreads();
    // s = r - alpha v
    run = __builtin_amdgcn_readfirstlane(L.run);
#pragma unroll
    for (int g = 0; g < G; ++g) m1[g] = own(DINV, g);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (!(run >> g & 1)) continue;
      r[g] = cfnma(L.alpha[g], at_v(g), r[g]);
      if (has) publish(gs, pub(1, turn, g), fresh(at_row), cmul(m1[g], r[g]));
    }
    {
      double none[1] = {0};
      if (group_sum<1, NT>(gs, B.size, rank, epoch, false, none, s_sums)) return;
    }
    // t = A D^-1 s; tau = t^H t, t^H s, ||s||^2
#pragma unroll 1
    for (int g = 0; g < slots; ++g)
      if (run >> g & 1) at_t(g) = product(pub(1, turn, g), L.kap[g]);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (g >= slots) continue;
      double sums[4] = {0, 0, 0, 0};
      if (run >> g & 1) {
        const V t = at_t(g);
        sums[0] = nrm2d(t);
        dotc_acc(t, r[g], sums[1], sums[2]);
        sums[3] = nrm2d(r[g]);
      }
      put(four, g, sums);
    }
    if (group_sum_wide<NP, NT>(gs, wide, B.size, rank, wepoch, 4 * slots, s_waves, s_parts)) return;
    if (w == 0) {
      const int g = lane;
      if (run >> g & 1 && g < G) {
        const double tau = total(0, 4, g), re = total(1, 4, g), im = total(2, 4, g), ss = total(3, 4, g);
        const bool half = isfinite(ss) && ss <= L.theta2[g];
        L.ss[g] = ss;
        if (!half && (!isfinite(ss) || !isfinite(tau) || !isfinite(re) || !isfinite(im))) {
          L.status[g] = HK_NONFINITE;
          L.done[g] = L.it[g] - 1;
        } else if (half || tau == 0) {
          L.status[g] = half ? S_HALF : S_TAUBD;
        } else {
          L.omega[g] = make_double2(re / tau, im / tau);
        }
      }
      masks(lane);
    }
    __syncthreads();
    // y += alpha p + omega s, r = s - omega t
    run = __builtin_amdgcn_readfirstlane(L.run);
    const unsigned half = __builtin_amdgcn_readfirstlane(L.half);
#pragma unroll
    for (int g = 0; g < G; ++g) m1[g] = own(RHAT, g);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (g >= slots) continue;
      double sums[4] = {0, 0, 0, 0};
      if ((run | half) >> g & 1) {
        V y = cfma(L.alpha[g], p[g], at_y(g));
        if (run >> g & 1) {
          const V om = L.omega[g];
          y = cfma(om, r[g], y);
          r[g] = cfnma(om, at_t(g), r[g]);
          sums[0] = nrm2d(r[g]);
          dotc_acc(m1[g], r[g], sums[1], sums[2]);
        }
        at_y(g) = y;
      }
      put(three, g, sums);
    }
    if (group_sum_wide<NP, NT>(gs, wide, B.size, rank, wepoch, 3 * slots, s_waves, s_parts)) return;
    if (w == 0) {
      const int g = lane;
      if (half >> g & 1 && g < G) {
        L.rr[g] = L.ss[g];
        L.done[g] = L.it[g];
        if (L.status[g] == S_TAUBD) L.bd[g] = HK_BD_TAU;
        L.status[g] = L.status[g] == S_HALF ? HK_OK : HK_BREAKDOWN;
      } else if (run >> g & 1 && g < G) {
        const double rr = total(0, 3, g);
        const V rho1 = make_double2(total(1, 3, g), total(2, 3, g)), om = L.omega[g];
        L.rr[g] = rr;
        L.done[g] = L.it[g];
        if (!isfinite(rr) || !cfinite(rho1)) {
          L.status[g] = HK_NONFINITE;
        } else if (rr <= L.theta2[g]) {
          L.status[g] = HK_OK;
        } else if (om.x == 0 && om.y == 0) {
          L.status[g] = HK_BREAKDOWN;
          L.bd[g] = HK_BD_OMEGA;
        } else if (rho1.x == 0 && rho1.y == 0) {
          L.status[g] = HK_BREAKDOWN;
          L.bd[g] = HK_BD_RHO;
        } else if (L.it[g] >= A.maxit) {
          L.status[g] = HK_NOT_CONVERGED;
        } else {
          L.beta[g] = cmul(cdiv(rho1, L.rho[g]), cdiv(L.alpha[g], om));
          L.rho[g] = rho1;
          ++L.it[g];
        }
      }
      masks(lane);
    }
    __syncthreads();
  }
}

const void* resident_many_kernel(const ResSweepPlan& p) {
  if (p.entries != 15) return nullptr;
  const bool local = p.span < p.grid;
  if (p.slots <= 3)
    return local ? (const void*)k_res_sweep_many<15, 3, 512, true> : (const void*)k_res_sweep_many<15, 3, 512, false>;
  return local ? (const void*)k_res_sweep_many<15, 6, 512, true> : (const void*)k_res_sweep_many<15, 6, 512, false>;
}
size_t resident_many_words(int slots) { return slots <= 3 ? WideSum<8>::kWords : WideSum<16>::kWords; }

}  // namespace hk
