// Kernels around the deterministic messenger iteration (the Wiener filter of
// the messenger scheme: the Gibbs sweep with every unit normal set to zero and
// P held fixed) and its adjoint.
//
// One iteration maps s_k to s_{k+1} = C (alpha s_k + beta), with
// C = F^-1 diag(f) F, f_b = P_b / (P_b + tau) per |k| bin, f = 0 at k = 0,
// alpha = 1 - tau R_i^2/N_i and beta = tau R_i d_i / N_i on observed voxels,
// (1, 0) elsewhere (Sec. 3.1: the means of the messenger and signal
// conditionals).  With R = 1 the loss is chi2_K = sum_i w_i d_i (d_i - s_K,i),
// w_i = 1/N_i (0 where unobserved), which tends to d^T (S + N)^-1 d as K
// grows; a response is handled by rescaling d to d / R.
//
// The sweep kernels run the iteration in deterministic modes (kZDet, kXDet,
// kXAdj, kPkGrad).  The kernels here build the iteration's inputs and finish
// its outputs; all of them walk the z-pass coefficient order, entry
// ((tile EPT + e) NT + tid) covering voxels (ix, iya, n) and (ix, iya + 1, n).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sweep_kernels.hpp"

namespace mf {

constexpr int kWienerThreads = 256;

template <typename R, int N>
__device__ __forceinline__ void entry_voxels(size_t idx, size_t& va, size_t& vb) {
  using T = ZTile<R, N>;
  const int tile = static_cast<int>(idx / (static_cast<size_t>(T::EPT) * T::NT));
  const int rem = static_cast<int>(idx % (static_cast<size_t>(T::EPT) * T::NT));
  int ix = 0, iya = 0, n = 0;
  zpass_coef_voxel<R, N>(tile, rem / T::NT, rem % T::NT, ix, iya, n);
  va = (static_cast<size_t>(ix) * N + iya) * N + n;
  vb = va + N;
}

// wcoef = (alpha_a, alpha_b, o_a d_a, o_b d_b): the messenger coefficients
// of the problem's noise model with new data d (FP64, [ix][iy][iz]); beta =
// tau d / N = o d with o = tau / N = 1 - alpha (with R = 1, after the
// rescaling by R).  o comes from the problem's own array (formed in FP64 and
// rounded once), not from 1 - alpha: in FP32, 1 - alpha would lose the
// relative precision 6e-8 N / tau where tau << N.
template <typename R, int N>
__global__ void __launch_bounds__(kWienerThreads)
wiener_coef_kernel(const R* coef, const R* omw, R* wcoef, const double* d, size_t entries) {
  const size_t idx = static_cast<size_t>(blockIdx.x) * kWienerThreads + threadIdx.x;
  if (idx >= entries) return;
  size_t va = 0, vb = 0;
  entry_voxels<R, N>(idx, va, vb);
  wcoef[idx * 4] = coef[idx * 4];
  wcoef[idx * 4 + 1] = coef[idx * 4 + 1];
  wcoef[idx * 4 + 2] = static_cast<R>(static_cast<double>(omw[idx * 2]) * d[va]);
  wcoef[idx * 4 + 3] = static_cast<R>(static_cast<double>(omw[idx * 2 + 1]) * d[vb]);
}

// Grid-unit P (P / V_cell) and the filter table (A_b = f_b / M, B_b unused).
template <typename R>
__global__ void wiener_table_kernel(const double* pk, double* pkg, R* table, double tau,
                                    double vcell, double m, int nb) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nb) return;
  const double p = pk[b] / vcell;
  pkg[b] = p;
  const double f = p / (p + tau);
  table[2 * b] = static_cast<R>(f / m);
  table[2 * b + 1] = R(0);
}

// y = x * w element by element (y may be x).  With w = 1 / R (0 where
// unobserved) it maps data d to d / R, and a gradient with respect to d / R
// to one with respect to d.
__global__ void scale_kernel(const double* x, const double* w, double* y, size_t n) {
  for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<size_t>(gridDim.x) * blockDim.x)
    y[i] = x[i] * w[i];
}

// Probe coefficients of the log-determinant estimator: (alpha, beta_z) with
// beta_z = tau R z / N for the probe z = sgn(R) sqrt(N) xi, i.e.
// beta_z = sqrt(tau o) xi with o = tau R^2 / N = 1 - alpha.  xi = +-1
// of voxel v comes from Philox counter (v div 4, probe, kPhaseProbe, chain),
// word v mod 4, top bit set -> -1.
template <typename R, int N>
__global__ void __launch_bounds__(kWienerThreads)
probe_coef_kernel(const R* coef, const R* omw, R* wcoef, double tau, uint32_t probe,
                  uint32_t chain, uint32_t k0, uint32_t k1, size_t entries) {
  const size_t idx = static_cast<size_t>(blockIdx.x) * kWienerThreads + threadIdx.x;
  if (idx >= entries) return;
  size_t va = 0, vb = 0;
  entry_voxels<R, N>(idx, va, vb);
  auto sign = [&](size_t v) {
    const Words4 w = philox4x32_10(static_cast<uint32_t>(v >> 2), probe, kPhaseProbe, chain, k0, k1);
    const uint32_t x = (v & 3) == 0 ? w.x0 : (v & 3) == 1 ? w.x1 : (v & 3) == 2 ? w.x2 : w.x3;
    return (x >> 31) ? -1.0 : 1.0;
  };
  wcoef[idx * 4] = coef[idx * 4];
  wcoef[idx * 4 + 1] = coef[idx * 4 + 1];
  wcoef[idx * 4 + 2] = static_cast<R>(sqrt(tau * static_cast<double>(omw[idx * 2])) * sign(va));
  wcoef[idx * 4 + 3] = static_cast<R>(sqrt(tau * static_cast<double>(omw[idx * 2 + 1])) * sign(vb));
}

// out_b += scale (G1_b - f_b G0_b) / (tau^2 V_cell), f_b = P_b / (P_b + tau):
// one probe's estimate of tr(A^-1 R S_b R) per unit of physical P_b, from the
// bin sums G1 = (1/M) sum Re(conj(t^_K) b^) and G0 = the same with t_{K-1}
// (b^ the transform of beta_z; s^_K = f t^_{K-1}).
__global__ void logdet_combine_kernel(const double* g1, const double* g0, const double* pkg,
                                      double tau, double vcell, double scale, int nb, double* out) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nb) return;
  const double f = pkg[b] / (pkg[b] + tau);
  out[b] += scale * (g1[b] - f * g0[b]) / (tau * tau * vcell);
}

template <typename T>
__global__ void fill_zero_kernel(T* p, size_t n) {
  for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<size_t>(gridDim.x) * blockDim.x)
    p[i] = T(0);
}

// Fixed-order block sum of kWienerThreads doubles in LDS; returns it on lane 0.
__device__ __forceinline__ double block_sum(double* red, double x) {
  const int tid = threadIdx.x;
  red[tid] = x;
  __syncthreads();
  for (int h = kWienerThreads / 2; h > 0; h >>= 1) {
    if (tid < h) red[tid] += red[tid + h];
    __syncthreads();
  }
  return red[0];
}

// Per-block partial sums of chi2 = sum_i w_i d_i (d_i - s_i), w = o / tau =
// 1 / N (0 where unobserved); optionally s_out = s (FP64, [ix][iy][iz]).  s
// is the iterate in [ix][iy][iz] order (the z-pass state read-out).
template <typename R, int N>
__global__ void __launch_bounds__(kWienerThreads)
wiener_chi2_kernel(const R* omw, const double* d, const R* s, double tau, double* partial,
                   double* s_out, size_t entries) {
  __shared__ double red[kWienerThreads];
  const size_t idx = static_cast<size_t>(blockIdx.x) * kWienerThreads + threadIdx.x;
  double x = 0.0;
  if (idx < entries) {
    size_t va = 0, vb = 0;
    entry_voxels<R, N>(idx, va, vb);
    const double wa = static_cast<double>(omw[idx * 2]) / tau;
    const double wb = static_cast<double>(omw[idx * 2 + 1]) / tau;
    const double sa = s[va], sb = s[vb];
    if (wa > 0.0) x += wa * d[va] * (d[va] - sa);
    if (wb > 0.0) x += wb * d[vb] * (d[vb] - sb);
    if (s_out) {
      s_out[va] = sa;
      s_out[vb] = sb;
    }
  }
  const double t = block_sum(red, x);
  if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// out[0] = sum of n partials in a fixed order (one workgroup).
__global__ void __launch_bounds__(kWienerThreads)
sum_partials_kernel(const double* partial, int n, double* out) {
  __shared__ double red[kWienerThreads];
  double x = 0.0;
  for (int i = threadIdx.x; i < n; i += kWienerThreads) x += partial[i];
  const double t = block_sum(red, x);
  if (threadIdx.x == 0) out[0] = t;
}

// d chi2 / d d_i = w_i (2 d_i - s_K,i) + o_i sum_k r_k,i (o = 1 - alpha), where
// r_k is the adjoint field; zero on unobserved voxels.  The direct term is
// written once s_K is known, the adjoint sum (acc, z-pass order) added last.
template <typename R, int N>
__global__ void __launch_bounds__(kWienerThreads)
wiener_grad_direct_kernel(const R* omw, const double* d, const R* s, double tau, double* grad_d,
                          size_t entries) {
  const size_t idx = static_cast<size_t>(blockIdx.x) * kWienerThreads + threadIdx.x;
  if (idx >= entries) return;
  size_t va = 0, vb = 0;
  entry_voxels<R, N>(idx, va, vb);
  const double oa = static_cast<double>(omw[idx * 2]);
  const double ob = static_cast<double>(omw[idx * 2 + 1]);
  grad_d[va] = oa / tau * (2.0 * d[va] - s[va]);
  grad_d[vb] = ob / tau * (2.0 * d[vb] - s[vb]);
}

template <typename R, int N>
__global__ void __launch_bounds__(kWienerThreads)
wiener_grad_adjoint_kernel(const R* omw, const R* acc, double* grad_d, size_t entries) {
  const size_t idx = static_cast<size_t>(blockIdx.x) * kWienerThreads + threadIdx.x;
  if (idx >= entries) return;
  size_t va = 0, vb = 0;
  entry_voxels<R, N>(idx, va, vb);
  grad_d[va] += static_cast<double>(omw[idx * 2]) * static_cast<double>(acc[idx * 2]);
  grad_d[vb] += static_cast<double>(omw[idx * 2 + 1]) * static_cast<double>(acc[idx * 2 + 1]);
}

// d chi2 / d P_b (physical units) = d chi2 / d f_b * tau / (P_b + tau)^2 / V_cell.
__global__ void wiener_grad_pk_kernel(const double* gacc, const double* pkg, double tau,
                                      double vcell, int nb, double* grad_pk) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nb) return;
  const double den = pkg[b] + tau;
  grad_pk[b] = gacc[b] * tau / (den * den) / vcell;
}

// ---------------------------------------------------------------- diagnostics
// Posterior mean and variance (population form, M2 / K) of a chain's recorded
// samples, from the z-pass-order Welford sums to [ix][iy][iz].  One workgroup
// per (z tile, element): its entries are QN neighbouring iz of every row of the
// tile, turned through LDS so that the stores are runs along iz (128 B at
// 256^3; stored from the entry order they were single values N rows apart).
// 256^3: 184 -> 106 us.
template <typename R, int N>
__global__ void __launch_bounds__((ZTile<R, N>::NT))
moments_kernel(const double* mom, double count, double* mean_out, double* var_out, size_t m) {
  using T = ZTile<R, N>;
  // at N = 8 a thread holds two pencils, and an entry's element half of them
  constexpr int PENS = T::NT < T::NPEN ? T::NT : T::NPEN;
  constexpr int QN = T::NT / PENS, ROWS = 2 * PENS, STR = QN + 1;
  __shared__ double mean_s[ROWS * STR], var_s[ROWS * STR];
  const int tid = threadIdx.x, tile = blockIdx.x / T::EPT, e = blockIdx.x % T::EPT;
  const size_t i = (static_cast<size_t>(blockIdx.x) * T::NT + tid) * 2;
  const int at = tid % PENS * 2 * STR + tid / PENS;
  mean_s[at] = mom[i];
  mean_s[at + STR] = mom[i + 1];
  var_s[at] = mom[m + i] / count;
  var_s[at + STR] = mom[m + i + 1] / count;
  __syncthreads();
  int ix = 0, iya = 0, n0 = 0;
  zpass_coef_voxel<R, N>(tile, e, 0, ix, iya, n0);   // the tile's first row, the first of its iz
  for (int it = tid; it < ROWS * QN; it += T::NT) {
    const int row = it / QN, q = it % QN;            // row = ix of the tile, then iy
    const size_t v = (static_cast<size_t>(ix + row / T::P) * N + iya + row % T::P) * N + n0 + q;
    mean_out[v] = mean_s[row * STR + q];
    var_out[v] = var_s[row * STR + q];
  }
}

// Autocorrelation of a recorded chain (Sec. 5.1, Eq. CORR_COEFF) of trace
// [t][nb]: with mean mu and variance var over the t samples of a bin,
// acf[n][b] = sum_{i < t-n} (x_i - mu)(x_{i+n} - mu) / ((t - n) var), n <=
// max_lag.
//
// t nb (max_lag + 1) FP64 products against t nb samples: bound by the FP64
// units once enough workgroups share the work, so a workgroup takes kAcfBins
// neighbouring bins (64 B of every trace row) and kAcfLags lags and walks the
// whole series in tiles of kAcfRows rows, the next tile's loads in flight
// during the products of this one.  The 64 threads of a bin each hold kAcfRun
// consecutive rows and the kAcfRun + kAcfLags - 1 later rows their lags need:
// 39 LDS reads for 128 products (254 VGPRs and 14 spilled outside the products).  An LDS run of 16 is padded to 17, which puts
// the 32 threads of a bin on different banks.  All sums run in a fixed order.
// 8000 samples of 32 bins, 400 lags: 46.5 us a call; one workgroup per bin and
// whole lags per thread, read from memory, took 2,320 us.  The series is walked
// tile by tile, and each tile costs one load latency: 512 rows by 256 threads
// take 55.8 us, 256 rows 99 us, and loads under a condition 115 us.
constexpr int kAcfThreads = 512, kAcfBins = 8, kAcfLags = 8, kAcfRun = 16, kAcfRows = 1024;
constexpr int kAcfPad = kAcfRows / kAcfRun * (kAcfRun + 1);   // padded rows of one bin
static_assert(kAcfThreads == kAcfBins * (kAcfRows / kAcfRun), "one run of rows per thread");
static_assert(kAcfThreads / kAcfBins == 64, "one wave per bin");

__global__ void __launch_bounds__(kAcfThreads)
acf_kernel(const double* trace, int t, int nb, int max_lag, int64_t items, double* acf) {
  constexpr int ROWS_PER_LOAD = kAcfThreads / kAcfBins;   // 64
  constexpr int LOADS = kAcfRows / ROWS_PER_LOAD;            // 16
  constexpr int S = kAcfPad + kAcfRun + 1;                   // one more run of later rows
  __shared__ double xa[kAcfBins * S], xw[kAcfBins * S];
  __shared__ double red[kAcfThreads];
  const int tid = threadIdx.x;
  const int lrow = tid / kAcfBins, lbin = tid % kAcfBins;    // this thread's loads
  const int cbin = tid / ROWS_PER_LOAD, run = tid % ROWS_PER_LOAD;   // this thread's products
  const int groups = (nb + kAcfBins - 1) / kAcfBins;
  // item = (lags, bins), bins fastest: neighbours share the trace's cache lines
  for (int64_t item = blockIdx.x; item < items; item += gridDim.x) {
    const int b0 = static_cast<int>(item % groups) * kAcfBins;
    const int n0 = static_cast<int>(item / groups) * kAcfLags;
    const double* col = trace + min(b0 + lbin, nb - 1);   // a bin past the last is never written
    // Rows past the end are loaded as the last row and replaced by 0 where they
    // are used: loads under a condition would be waited for one by one.
    auto row_at = [&](int64_t i) { return col[static_cast<size_t>(min(i, static_cast<int64_t>(t) - 1)) * nb]; };
    // mean of every bin, counted from its first sample so that the mean of a
    // constant series is that sample exactly: 64 strided sums, added in order
    const double x0 = col[0];
    double sum = 0.0;
    constexpr int MEAN_ROWS = 32 * ROWS_PER_LOAD;
    int64_t im = 0;
    for (; im + MEAN_ROWS <= t; im += MEAN_ROWS) {
      double x[32];
#pragma unroll
      for (int k = 0; k < 32; ++k) x[k] = col[static_cast<size_t>(im + lrow + k * ROWS_PER_LOAD) * nb];
#pragma unroll
      for (int k = 0; k < 32; ++k) sum += x[k] - x0;
    }
    if (im < t) {
      double x[32];
#pragma unroll
      for (int k = 0; k < 32; ++k) x[k] = row_at(im + lrow + k * ROWS_PER_LOAD);
#pragma unroll
      for (int k = 0; k < 32; ++k) sum += im + lrow + k * ROWS_PER_LOAD < t ? x[k] - x0 : 0.0;
    }
    red[tid] = sum;
    __syncthreads();
    double mu = 0.0;
    for (int r = 0; r < ROWS_PER_LOAD; ++r) mu += red[r * kAcfBins + lbin];
    mu = x0 + mu / t;
    auto slot = [](int row) { return row + row / kAcfRun; };
    double acc[kAcfLags] = {0.0}, sq = 0.0;
    double pa[LOADS], pw[LOADS + 1];
    auto fetch = [&](int64_t i0) {
#pragma unroll
      for (int k = 0; k < LOADS; ++k) {
        const int64_t i = i0 + lrow + k * ROWS_PER_LOAD;
        pa[k] = row_at(i);
        pw[k] = row_at(i + n0);
      }
      pw[LOADS] = row_at(i0 + n0 + kAcfRows + lrow);
    };
    fetch(0);
    for (int64_t i0 = 0; i0 < t; i0 += kAcfRows) {
      __syncthreads();   // the previous tile is used up
#pragma unroll
      for (int k = 0; k < LOADS; ++k) {
        const int64_t i = i0 + lrow + k * ROWS_PER_LOAD;
        xa[lbin * S + slot(lrow + k * ROWS_PER_LOAD)] = i < t ? pa[k] - mu : 0.0;
        xw[lbin * S + slot(lrow + k * ROWS_PER_LOAD)] = i + n0 < t ? pw[k] - mu : 0.0;
      }
      if (lrow < kAcfRun)
        xw[lbin * S + slot(kAcfRows + lrow)] = i0 + n0 + kAcfRows + lrow < t ? pw[LOADS] - mu : 0.0;
      __syncthreads();
      if (i0 + kAcfRows < t) fetch(i0 + kAcfRows);
      double x[kAcfRun], w[kAcfRun + kAcfLags - 1];
#pragma unroll
      for (int r = 0; r < kAcfRun; ++r) x[r] = xa[cbin * S + run * (kAcfRun + 1) + r];
#pragma unroll
      for (int r = 0; r < kAcfRun + kAcfLags - 1; ++r)
        w[r] = xw[cbin * S + run * (kAcfRun + 1) + r + r / kAcfRun];
#pragma unroll
      for (int r = 0; r < kAcfRun; ++r) {
        sq += x[r] * x[r];
#pragma unroll
        for (int j = 0; j < kAcfLags; ++j) acc[j] += x[r] * w[r + j];
      }
    }
#pragma unroll
    for (int h = ROWS_PER_LOAD / 2; h > 0; h >>= 1) {
      sq += __shfl_xor(sq, h);
#pragma unroll
      for (int j = 0; j < kAcfLags; ++j) acc[j] += __shfl_xor(acc[j], h);
    }
    if (run == 0 && b0 + cbin < nb) {
      const double var = sq / t;
#pragma unroll
      for (int j = 0; j < kAcfLags; ++j) {
        const int n = n0 + j;
        if (n <= max_lag)
          acf[static_cast<size_t>(n) * nb + b0 + cbin] = acc[j] / ((t - n) * var);
      }
    }
  }
}

// First lag with acf < 0.1 of bin b, -1 if none, by one wave.
__device__ __forceinline__ void acf_length(const double* acf, int nb, int max_lag, int b, int lane, int32_t* nc) {
  for (int n0 = 0; n0 <= max_lag; n0 += 64) {
    const int n = n0 + lane;
    const bool low = n <= max_lag && acf[static_cast<size_t>(n) * nb + b] < 0.1;
    const unsigned long long m = __ballot(low);
    if (m != 0) {
      if (lane == 0) nc[b] = n0 + __ffsll(m) - 1;
      return;
    }
  }
  if (lane == 0) nc[b] = -1;
}

// Short series: one workgroup per bin holds all of it in LDS, takes a lag per
// thread in turn and finds the length in the same launch.  Tiles would be mostly
// empty, and each workgroup of them takes some 7 us.  A call, tiles : this, 50
// samples of 5 bins and 10 lags 14.7 : 11.4 us, 100 of 200 and 99 lags 26.2 :
// 11.5, 300 of 8 and 15 lags 15.2 : 12.8; but 384 of 16 and 30 lags 14.8 : 15.4.
constexpr int kAcfShort = 320, kAcfShortThreads = kWienerThreads;

__global__ void __launch_bounds__(kAcfShortThreads)
acf_short_kernel(const double* trace, int t, int nb, int max_lag, double* acf, int32_t* nc) {
  __shared__ double x[kAcfShort + 8], red[kAcfShortThreads], sums[kAcfShort];
  const int b = blockIdx.x, tid = threadIdx.x;
  const double x0 = trace[b];   // the mean counted from it, as in acf_kernel
  double s = 0.0;
  for (int i = tid; i < t + 8; i += kAcfShortThreads) {
    x[i] = i < t ? trace[static_cast<size_t>(i) * nb + b] : 0.0;
    if (i < t) s += x[i] - x0;
  }
  const double mu = x0 + block_sum(red, s) / t;
  __syncthreads();
  for (int i = tid; i < t; i += kAcfShortThreads) x[i] -= mu;
  __syncthreads();
  for (int n = tid; n <= max_lag; n += kAcfShortThreads) {
    double acc[8] = {0.0};
    for (int i = 0; i < t - n; i += 8)
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[k] += x[i + k] * (i + k < t - n ? x[i + k + n] : 0.0);
    sums[n] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
  }
  __syncthreads();
  const double var = sums[0] / t;
  for (int n = tid; n <= max_lag; n += kAcfShortThreads)
    acf[static_cast<size_t>(n) * nb + b] = sums[n] / ((t - n) * var);
  __syncthreads();
  if (tid < 64) acf_length(acf, nb, max_lag, b, tid, nc);
}

// The lengths after acf_kernel: one wave per bin.
__global__ void __launch_bounds__(64)
acf_length_kernel(const double* acf, int nb, int max_lag, int32_t* nc) {
  acf_length(acf, nb, max_lag, blockIdx.x, threadIdx.x, nc);
}

}  // namespace mf
