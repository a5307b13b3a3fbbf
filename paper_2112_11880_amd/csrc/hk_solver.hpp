// hk_solver.hpp -- scalar state and helpers shared by the plain solvers' kernels
// (hk_solver.hip) and the resident ones (hk_resident.hip).
#pragma once

#include "hk_common.hpp"
#include "hk_internal.hpp"

namespace hk {

// Transient statuses (>= S_RUN): the solve goes on, or an exit is pending
// until the kernels of the current iteration have applied their last update.
enum : int { S_RUN = 100, S_HALF = 101, S_TAUBD = 102, S_HALF2 = 103, S_RHOBD = 104 };

struct SolveState {
  double2 rho, rho_old, alpha, omega, beta;
  double rr, ss, bb, theta2, rr_true;
  int status, bd;
  long long iter, maxit, iters_done;
  double* history;
  // TFQMR: theta, tau, the two half-steps' eta (their x updates are applied
  // by the next kernel that reads d) and the d-update coefficients
  double tq_theta, tq_tau;
  double2 tq_eta1, tq_eta2, tq_coef1, tq_coef2;
  // BiCGStab(l): the minimal-residual coefficients gamma_1..gamma_l
  double2 bl_gamma[8];
};

// a solver scalar (double) rounded to the vector type
template <class V> __device__ __forceinline__ V vscal(double2 a) {
  return cmake<V>((decltype(V::x))a.x, (decltype(V::x))a.y);
}
// |a|^2 in double
template <class V> __device__ __forceinline__ double nrm2d(V a) {
  const double x = a.x, y = a.y;
  return x * x + y * y;
}
// acc += conj(a) * b in double (two partial sums: re, im)
template <class V> __device__ __forceinline__ void dotc_acc(V a, V b, double& re, double& im) {
  const double ax = a.x, ay = a.y, bx = b.x, by = b.y;
  re = fma(ax, bx, fma(ay, by, re));
  im = fma(ax, by, fma(-ay, bx, im));
}

}  // namespace hk
