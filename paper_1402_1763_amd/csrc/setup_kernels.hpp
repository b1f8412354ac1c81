// Set-up of a problem from the caller's FP64 arrays (noise variance N, response
// R, data d), staged on the device: a chain's messenger coefficients in the
// z-pass order.  Every value is formed by the FP64 operations of the messenger
// conditional in one fixed order (correctly rounded divisions included), so it
// is the same wherever it is formed.
//
// Bound by the copies from pageable host memory (16 B a voxel at some 25 GB/s).
// The whole set-up of a 128^3 FP32 problem takes 3.6 ms, of 256^3 25.8 ms; with
// the coefficients formed and permuted on the host (and the bins counted mode
// by mode) it took 13.4 and 135 ms.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sweep_kernels.hpp"

namespace mf {

constexpr int kSetupThreads = 256;

__device__ __forceinline__ bool voxel_observed(double noise, double resp) {
  return !isinf(noise) && resp != 0.0;
}

// Messenger coefficients of Sec. 3.1 with T = tau and N~ = N - tau R^2:
// mean = alpha s + beta with alpha = N~ / N = 1 - tau R^2 / N and
// beta = tau R d / N; (1, 0) where unobserved.  alpha is 0 in exact
// arithmetic where N / R^2 is smallest (tau is that minimum); rounding of
// tau R^2 / N there can leave -1 ulp, which is set back to 0.
// Also o = tau R^2 / N (0 where unobserved) per voxel, entry order
// [entry][2], for the Wiener filter's data-dependent coefficients.
// noise, resp and data hold the voxels from voxel0 on, a whole number of z-pass
// tiles: the entries entry0 .. entry0 + entries - 1.  One workgroup covers
// neighbouring entries, so its loads are short runs along z of a few pencils,
// which the caches put together; the stores are whole lines.
template <typename R, int N>
__global__ void __launch_bounds__(kSetupThreads)
setup_coef_kernel(const double* noise, const double* resp, const double* data, double tau,
                  size_t voxel0, size_t entry0, size_t entries, R* coef, R* omw, uint32_t* obs) {
  using T = ZTile<R, N>;
  const size_t k = static_cast<size_t>(blockIdx.x) * kSetupThreads + threadIdx.x;
  if (k >= entries) return;
  const size_t idx = entry0 + k;
  const int tile = static_cast<int>(idx / (static_cast<size_t>(T::EPT) * T::NT));
  const int rem = static_cast<int>(idx % (static_cast<size_t>(T::EPT) * T::NT));
  const int e = rem / T::NT;
  int ix = 0, iya = 0, n = 0;
  zpass_coef_voxel<R, N>(tile, e, rem % T::NT, ix, iya, n);
  const size_t va = (static_cast<size_t>(ix) * N + iya) * N + n - voxel0;
  bool any = false;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const size_t i = va + h * N;
    const double nv = noise[i], r = resp ? resp[i] : 1.0, d = data[i];
    const bool seen = voxel_observed(nv, r);
    const double o = tau * r * r / nv;
    coef[idx * 4 + h] = static_cast<R>(seen ? fmax(0.0, 1.0 - o) : 1.0);
    coef[idx * 4 + 2 + h] = static_cast<R>(seen ? tau * r * d / nv : 0.0);
    omw[idx * 2 + h] = static_cast<R>(seen ? fmin(1.0, o) : 0.0);
    any |= seen;
  }
  // one atomic per wave where its lanes share the tile and the element
  const int key = tile * 32 + e, first = __builtin_amdgcn_readfirstlane(key);
  if (__all(key == first)) any = __any(any) && __ffsll(__ballot(true)) - 1 == static_cast<int>(threadIdx.x % 64);
  if (any) atomicOr(obs + tile, 1u << e);
}

// 1 / R per voxel (0 where unobserved), in place over R.
__global__ void __launch_bounds__(kSetupThreads)
setup_rinv_kernel(const double* noise, double* resp, size_t m) {
  for (size_t i = static_cast<size_t>(blockIdx.x) * kSetupThreads + threadIdx.x; i < m;
       i += static_cast<size_t>(gridDim.x) * kSetupThreads) {
    const double r = resp[i];
    resp[i] = voxel_observed(noise[i], r) ? 1.0 / r : 0.0;
  }
}

}  // namespace mf
