// hk_slice.hip -- slices of a matrix: their distances, their values (gfx950).
#include <climits>
#include <vector>

#include "hk_slice.hpp"

namespace hk {

// The slices read 16 bytes per value where the row blocks read 18 and the row
// pointers, and go without the LDS: up to this many values per entry they were
// faster throughout (a BiCGStab iteration, slices against row blocks: 1.03 values
// per entry 257 and 290 us on 1.8M rows; flat boxes of 160 to 350 thousand rows with
// 1.09 77 and 90, 1.17 71 and 84, 1.27 78.5 and 82.5).
constexpr double kSliceMost = 1.25;
constexpr int kSliceBlock = 4 * kWave;

// The distances of one slice, ascending: f(number, distance, this lane's row has
// it, its entry).  Returns how many.
template <class F>
__device__ __forceinline__ int slice_walk(int slice, int n, const int* rowptr, const int* col, F&& f) {
  const int l = threadIdx.x & (kWave - 1), r = slice * kWave + l;
  int p = r < n ? rowptr[r] : 0;
  const int e = r < n ? rowptr[r + 1] : 0;
  for (int j = 0;; ++j) {
    const int mine = p < e ? col[p] - r : INT_MAX;
    int least = mine;
#pragma unroll
    for (int d = kWave / 2; d > 0; d /= 2) least = min(least, __shfl_xor(least, d));
    if (least == INT_MAX) return j;
    const bool has = mine == least;
    f(j, least, has, p);
    if (has) ++p;
  }
}

// cnt[slice]: its distances
__global__ __launch_bounds__(kSliceBlock) void k_slice_count(int n, int nslices, const int* __restrict__ rowptr,
                                                             const int* __restrict__ col, int* __restrict__ cnt) {
  const int slice = (int)(blockIdx.x * (kSliceBlock / kWave) + threadIdx.x / kWave);
  if (slice >= nslices) return;
  const int c = slice_walk(slice, n, rowptr, col, [](int, int, bool, int) {});
  if ((threadIdx.x & (kWave - 1)) == 0) cnt[slice] = c;
}

__global__ __launch_bounds__(kSliceBlock) void k_slice_off(int n, int nslices, const int* __restrict__ rowptr,
                                                           const int* __restrict__ col, const int* __restrict__ ptr,
                                                           int* __restrict__ off) {
  const int slice = (int)(blockIdx.x * (kSliceBlock / kWave) + threadIdx.x / kWave);
  if (slice >= nslices) return;
  const int base = ptr[slice];
  slice_walk(slice, n, rowptr, col, [&](int j, int d, bool, int) {
    if ((threadIdx.x & (kWave - 1)) == 0) off[base + j] = d;
  });
}

template <class V>
__global__ __launch_bounds__(kSliceBlock) void k_slice_fill(int n, int nslices, const int* __restrict__ rowptr,
                                                            const int* __restrict__ col,
                                                            const int* __restrict__ ptr, const V* __restrict__ val,
                                                            const V* __restrict__ dinv, V* __restrict__ out) {
  const int slice = (int)(blockIdx.x * (kSliceBlock / kWave) + threadIdx.x / kWave);
  if (slice >= nslices) return;
  V* const o = out + (size_t)ptr[slice] * kWave + (threadIdx.x & (kWave - 1));
  slice_walk(slice, n, rowptr, col, [&](int j, int, bool has, int p) {
    V v = czero<V>();
    if (has) v = cmul(val[p], dinv[col[p]]);
    stnt(o + (size_t)j * kWave, v);
  });
}

static dim3 slice_grid(int nslices) { return dim3((unsigned)((nslices + kSliceBlock / kWave - 1) / (kSliceBlock / kWave))); }

int slices_prepare(hk_csr_s* A, hipStream_t s) {
  SliceStore& S = A->slices;
  if (S.tried || A->nnz <= 0) return HK_OK;
  S.tried = true;
  const int n = (int)A->n, ns = (n + kWave - 1) / kWave;
  std::vector<int> h(ns + 1);
  int* ptr = nullptr;
  if (hipMalloc(&ptr, sizeof(int) * (ns + 1)) != hipSuccess) {
    (void)hipGetLastError();  // the row blocks do without
    return HK_OK;
  }
  hipLaunchKernelGGL(k_slice_count, slice_grid(ns), dim3(kSliceBlock), 0, s, n, ns, A->rowptr, A->col, ptr);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpyAsync(h.data(), ptr, sizeof(int) * ns, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  long long sum = 0;
  for (int k = 0; k < ns && e == hipSuccess; ++k) {
    const int c = h[k];
    h[k] = (int)std::min<long long>(sum, INT_MAX);
    sum += c;
  }
  h[ns] = (int)std::min<long long>(sum, INT_MAX);
  int* off = nullptr;
  const bool fits = e == hipSuccess && sum > 0 && (double)sum * kWave <= kSliceMost * (double)A->nnz;
  if (fits && hipMalloc(&off, sizeof(int) * sum) == hipSuccess) {
    e = hipMemcpyAsync(ptr, h.data(), sizeof(int) * (ns + 1), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) {
      hipLaunchKernelGGL(k_slice_off, slice_grid(ns), dim3(kSliceBlock), 0, s, n, ns, A->rowptr, A->col, ptr, off);
      e = hipGetLastError();
    }
    const hipError_t se = hipStreamSynchronize(s);  // h lives on this frame
    if (e == hipSuccess) e = se;
  }
  if (e != hipSuccess || !off) {
    (void)hipFree(ptr);
    if (off) (void)hipFree(off);
    if (e != hipSuccess) HK_FAIL(HK_EHIP, "krylov solve: slices: %s", hipGetErrorString(e));
    (void)hipGetLastError();
    return HK_OK;
  }
  S.ptr = ptr;
  S.off = off;
  S.count = ns;
  S.values = sum * kWave;
  return HK_OK;
}

template <class V>
hipError_t slices_fill(const hk_csr_s* A, const V* val, const V* dinv, V* out, hipStream_t s) {
  hipLaunchKernelGGL(k_slice_fill<V>, slice_grid(A->slices.count), dim3(kSliceBlock), 0, s, (int)A->n, A->slices.count,
                     A->rowptr, A->col, A->slices.ptr, val, dinv, out);
  return hipGetLastError();
}
template hipError_t slices_fill<double2>(const hk_csr_s*, const double2*, const double2*, double2*, hipStream_t);
template hipError_t slices_fill<float2>(const hk_csr_s*, const float2*, const float2*, float2*, hipStream_t);

}  // namespace hk
