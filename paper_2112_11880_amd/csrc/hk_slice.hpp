// hk_slice.hpp -- the solvers' matrix in slices of 64 rows (gfx950).
//
// A mesh's rows hold their entries at few distinct distances col - row: 15 for
// tetrahedra and 27 for hexahedra numbered along a box.  A slice of 64
// consecutive rows keeps the distances that any of its rows has, ascending, and
// for each of them 64 values, zero where a row has no such entry.  A wave takes
// a slice, a lane a row: values and x are read 64 consecutive elements at a
// time, no column and no row pointer is read, and no product goes through LDS as
// in the row blocks of hk_spmv.hpp.  The values are the solver's own copy,
// A D^-1, laid out anew by every solve; the distances are the handle's.  Memory
// bounds it: 1,815,937 rows with 15 distances per slice are 523 MB for a fused
// product instead of the row blocks' 573, and a BiCGStab iteration takes 257 us
// instead of 290 (TFQMR 284 and 315), on 409,457 rows of 15 80 and 91, on 226,981
// of 27 71 and 85.
#pragma once

#include "hk_internal.hpp"
#include "hk_spmv.hpp"

namespace hk {

// SpmvPlan::L of the sliced products; U = 64, nw waves per workgroup.
constexpr int kSliceL = 2;
constexpr int kSliceWaves = 4;

// Sum of row 64 * slice + lane of values at val + 64 ptr[slice]: in the order of
// the columns, a step's five products added up by themselves (the first three in a
// chain), which keeps the sum of the row from being rounded at each entry: 1.65e-16
// of 15 entries on a random vector and 1.73e-16 of 27, no more than the row blocks of
// 32 and 16 rows that such systems had (one chain over the row: 2.7e-16 and
// 3.5e-16).  A BiCGStab iteration on 1.8M rows takes 253 us, as with one chain
// (252.7); a cut after the diagonal by scalar branches took 254.5.  complex64 in
// double, whose conversions are free beside the loads.  `ptr` and `off` are read by
// scalar loads.
template <class V>
__device__ __forceinline__ V slice_row(int slice, int n, const int* __restrict__ ptr, const int* __restrict__ off,
                                       const V* __restrict__ val, const V* __restrict__ x) {
  constexpr int U = 5;  // loads of 5 distances in flight
  const int l = threadIdx.x & (kWave - 1), r = min(slice * kWave + l, n - 1);
  int j = __builtin_amdgcn_readfirstlane(ptr[slice]);
  const int end = __builtin_amdgcn_readfirstlane(ptr[slice + 1]);
  double2 acc = make_double2(0, 0);
  auto col = [&](int d) { return min(max(r + d, 0), n - 1); };
  auto wide = [](V v) { return make_double2(v.x, v.y); };
  for (; j + U <= end; j += U) {
    V a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = ldnt(val + (size_t)(j + u) * kWave + l);
#pragma unroll
    for (int u = 0; u < U; ++u) b[u] = x[col(off[j + u])];
    double2 part = cmul(wide(a[0]), wide(b[0]));
    part = cfma(wide(a[1]), wide(b[1]), part);
    part = cfma(wide(a[2]), wide(b[2]), part);
#pragma unroll
    for (int u = 3; u < U; ++u) part = cadd(part, cmul(wide(a[u]), wide(b[u])));
    acc = cadd(acc, part);
  }
  double2 rest = make_double2(0, 0);
  for (; j < end; ++j) rest = cfma(wide(ldnt(val + (size_t)j * kWave + l)), wide(x[col(off[j])]), rest);
  acc = cadd(acc, rest);
  return cmake<V>((decltype(V::x))acc.x, (decltype(V::x))acc.y);
}

// Finds the slices of A's pattern and keeps them in the handle, once; leaves none
// there if they would hold more than kSliceMost values per entry.
int slices_prepare(hk_csr_s* A, hipStream_t s);
// A D^-1 in slices: val of A's entries, 64 values per distance in out.
template <class V>
hipError_t slices_fill(const hk_csr_s* A, const V* val, const V* dinv, V* out, hipStream_t s);

}  // namespace hk
