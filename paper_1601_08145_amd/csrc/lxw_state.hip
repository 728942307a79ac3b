// State transfer between the caller's layout Q[N][V][ML] (float64, caller's element order) and the
// solver's: cell averages Qbar[N][V] (float64) and higher modes Qh[V][ML-1][N] (bulk type), internal
// element order; and the check of a caller's state (lxw_set_state).
//
// Bound by HBM: a state is read once and written once.  Rows of the caller's array (V * ML values,
// 72 to 400 bytes) are read and written by consecutive lanes, columns of the solver's by consecutive
// elements; a tile of 64 elements is turned between the two in LDS (rows padded to an odd count of
// doubles, so that the column side meets no bank conflict).  Formerly the state went through host
// memory and two host loops: 161 ms in and 137 ms out for 999,698 triangles (24 values each) held in
// device memory; now 0.17 ms in (check and transfer, two reads of the state) and 0.11 ms out, calls
// whole.
#include <hip/hip_runtime.h>

#include "lxw_internal.hpp"

namespace lxw {

constexpr int TILE = 64, TPB = 256;

// Rows [c0, c1) of the caller's array start at Q; elements off .. off + n of the solver hold the
// caller's elements perm[off + i] - off.  Elements outside the rows at hand are left alone.
template <int ML, class R>
__global__ __launch_bounds__(TPB) void k_import(const double* Q, int c0, int c1, const int* perm, int off, int n, int V,
                                                int Nt, double* Qbar, R* Qh) {
  extern __shared__ double lds[];
  __shared__ int row[TILE];
  const int W = V * ML, S = W | 1;
  const int i0 = (int)blockIdx.x * TILE;
  const int m = min(TILE, n - i0);
  if ((int)threadIdx.x < m) {
    const int c = perm[off + i0 + threadIdx.x] - off;
    row[threadIdx.x] = (c >= c0 && c < c1) ? c - c0 : -1;
  }
  __syncthreads();
  for (int x = threadIdx.x; x < m * W; x += TPB) {
    const int e = x / W, w = x - e * W;
    if (row[e] >= 0) lds[e * S + w] = Q[(size_t)row[e] * W + w];
  }
  __syncthreads();
  for (int x = threadIdx.x; x < m * V; x += TPB) {
    const int e = x / V, c = x - e * V;
    if (row[e] >= 0) Qbar[(size_t)(off + i0 + e) * V + c] = lds[e * S + c * ML];
  }
  const int e = threadIdx.x & (TILE - 1);
  if (e < m && row[e] >= 0)
    for (int r = threadIdx.x / TILE; r < V * (ML - 1); r += TPB / TILE) {
      const int c = r / (ML - 1), l = r - c * (ML - 1);
      Qh[(size_t)r * Nt + off + i0 + e] = R(lds[e * S + c * ML + 1 + l]);
    }
}

template <int ML, class R>
__global__ __launch_bounds__(TPB) void k_export(double* Q, int c0, int c1, const int* perm, int off, int n, int V, int Nt,
                                                const double* Qbar, const R* Qh) {
  extern __shared__ double lds[];
  __shared__ int row[TILE];
  const int W = V * ML, S = W | 1;
  const int i0 = (int)blockIdx.x * TILE;
  const int m = min(TILE, n - i0);
  if ((int)threadIdx.x < m) {
    const int c = perm[off + i0 + threadIdx.x] - off;
    row[threadIdx.x] = (c >= c0 && c < c1) ? c - c0 : -1;
  }
  __syncthreads();
  for (int x = threadIdx.x; x < m * V; x += TPB) {
    const int e = x / V, c = x - e * V;
    if (row[e] >= 0) lds[e * S + c * ML] = Qbar[(size_t)(off + i0 + e) * V + c];
  }
  const int e0 = threadIdx.x & (TILE - 1);
  if (e0 < m && row[e0] >= 0)
    for (int r = threadIdx.x / TILE; r < V * (ML - 1); r += TPB / TILE) {
      const int c = r / (ML - 1), l = r - c * (ML - 1);
      lds[e0 * S + c * ML + 1 + l] = double(Qh[(size_t)r * Nt + off + i0 + e0]);
    }
  __syncthreads();
  for (int x = threadIdx.x; x < m * W; x += TPB) {
    const int e = x / W, w = x - e * W;
    if (row[e] >= 0) Q[(size_t)row[e] * W + w] = lds[e * S + w];
  }
}

// First element (caller's order) of rows [c0, c0 + n) whose average violates rho_bar >= eps0 or
// p_bar > 0, or that holds a value that is not finite: the minimum of c0 + index over them, into
// *bad.  One lane per value reads the rows; the products are rounded one by one (no fused
// multiply-adds), as the check on host data always was.
template <int ML>
__global__ __launch_bounds__(TPB) void k_check(const double* Q, int c0, int n, int V, double gm1, double eps0, int* bad) {
  extern __shared__ double lds[];
  __shared__ int fail[TILE];
  const int W = V * ML, S = V | 1;
  const int i0 = (int)blockIdx.x * TILE;
  const int m = min(TILE, n - i0);
  if (threadIdx.x < TILE) fail[threadIdx.x] = 0;
  __syncthreads();
  for (int x = threadIdx.x; x < m * W; x += TPB) {
    const int e = x / W, w = x - e * W;
    const double q = Q[(size_t)i0 * W + x];
    if (!isfinite(q)) fail[e] = 1;
    if (w % ML == 0) lds[e * S + w / ML] = q;
  }
  __syncthreads();
  const int e = threadIdx.x;
  if (e >= m) return;
  const double* qb = lds + e * S;
  double k = 0.0;
  for (int d = 1; d < V - 1; ++d) k = add_rn(k, mul_rn(qb[d], qb[d]));
  const double p = mul_rn(gm1, sub_rn(qb[V - 1], mul_rn(0.5, k) / qb[0]));
  if (fail[e] || !(qb[0] >= eps0) || !(p > 0.0)) atomicMin(bad, c0 + i0 + e);
}

// Calls f.template operator()<ML>() for the mode counts the elements have.
template <class F>
static hipError_t by_modes(int ML, F&& f) {
  switch (ML) {
    case 3: f(std::integral_constant<int, 3>()); break;
    case 4: f(std::integral_constant<int, 4>()); break;
    case 6: f(std::integral_constant<int, 6>()); break;
    case 9: f(std::integral_constant<int, 9>()); break;
    case 10: f(std::integral_constant<int, 10>()); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
static dim3 tiles(int n) { return dim3((unsigned)((n + TILE - 1) / TILE)); }

template <class R>
hipError_t launch_import(const double* Q, int c0, int c1, const int* perm, int off, int n, int V, int ML, int Nt,
                         double* Qbar, R* Qh, hipStream_t st) {
  if (n < 1) return hipSuccess;
  return by_modes(ML, [&](auto m) {
    hipLaunchKernelGGL((k_import<m(), R>), tiles(n), dim3(TPB), TILE * (V * ML | 1) * sizeof(double), st, Q, c0, c1, perm,
                       off, n, V, Nt, Qbar, Qh);
  });
}

template <class R>
hipError_t launch_export(double* Q, int c0, int c1, const int* perm, int off, int n, int V, int ML, int Nt,
                         const double* Qbar, const R* Qh, hipStream_t st) {
  if (n < 1) return hipSuccess;
  return by_modes(ML, [&](auto m) {
    hipLaunchKernelGGL((k_export<m(), R>), tiles(n), dim3(TPB), TILE * (V * ML | 1) * sizeof(double), st, Q, c0, c1, perm,
                       off, n, V, Nt, Qbar, Qh);
  });
}

hipError_t launch_check(const double* Q, int c0, int n, int V, int ML, double gm1, double eps0, int* bad, hipStream_t st) {
  if (n < 1) return hipSuccess;
  return by_modes(ML, [&](auto m) {
    hipLaunchKernelGGL((k_check<m()>), tiles(n), dim3(TPB), TILE * (V | 1) * sizeof(double), st, Q, c0, n, V, gm1, eps0,
                       bad);
  });
}

template hipError_t launch_import<double>(const double*, int, int, const int*, int, int, int, int, int, double*, double*, hipStream_t);
template hipError_t launch_import<float>(const double*, int, int, const int*, int, int, int, int, int, double*, float*, hipStream_t);
template hipError_t launch_export<double>(double*, int, int, const int*, int, int, int, int, int, const double*, const double*, hipStream_t);
template hipError_t launch_export<float>(double*, int, int, const int*, int, int, int, int, int, const double*, const float*, hipStream_t);

}  // namespace lxw
