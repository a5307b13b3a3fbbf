// hk_resident.hpp -- launch interface of the resident solves.
#pragma once

#include "hk_grid.hpp"
#include "hk_internal.hpp"
#include "hk_solver.hpp"

namespace hk {

template <class R> struct ResArgs {
  using V = cplx<R>;
  int n, rows;             // rows per workgroup: a multiple of 64
  const int* rowptr;
  const int* col;
  const V* val;
  const V* dinv;
  const V* b;
  const V* x0;             // null: start from 0; else r0 holds b - A x0
  const V* r0;
  V* y;                    // D x at the end
  V* pub[4];               // vectors the workgroups publish to each other
  SolveState* st;          // the solve's state at the end
  const int* flag;         // zero-diagonal flag of the set-up: nonzero ends the kernel
  GridSum gs;
  double tol;
  long long maxit;
  double* history;
};

// Enqueues the solve on s: barrier words, state, then the cooperative
// launch.  hipErrorInvalidConfiguration (or what the launch gave) if it
// cannot run here.
template <class R> hipError_t resident_launch(const ResShape& sh, int method, ResArgs<R> args, void* scratch,
                                              hipStream_t s);
// The abort flag in the scratch (device address).
int* resident_abort(void* scratch);

}  // namespace hk
