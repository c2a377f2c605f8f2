// Privacy accounting with an envelope CDF (appendix: Algorithm accounting and the
// binning of the envelope law that feeds it), fp64.
//
// * envelope_bins_kernel: the envelope law of Y as bins.  From F(y_0..y_M) on an
//   even grid it takes the running maximum (a CDF evaluated numerically may dip),
//   clips to [0, 1], takes the increments as bin weights, clamps them at zero,
//   normalises them to sum to one, and puts each bin's weight at its midpoint.
// * pld_survival_kernel: one subsampled step's privacy-loss survival function
//   S(t) = P(L > t) at the cut points t = (c - n + 1/2) h, c = 0 .. 2n - 1.  With
//   amplification by subsampling at rate p, S(t) = p betabar(t + s(t)) +
//   (1 - p) alpha(t + s(t)), s(t) = log(1/p - (1-p)/p e^-t), above the support
//   bound log(1 - p), and S = 1 at and below it.  alpha and betabar are the
//   Gaussian test errors at signal-to-noise mu = a / sigma averaged over the
//   envelope bins with a_i = 1 / sqrt(ybar_i) (or a = 1 without an envelope):
//   alpha(u) = sum_i w_i Phi(-u/mu_i - mu_i/2), betabar(u) = sum_i w_i Phi(-u/mu_i + mu_i/2).
//   A workgroup of eight waves takes 64 cut points; each wave sums its eighth of the bins
//   for all of them (a lane per cut, the bins' 1/mu and mu/2 computed once per wave), and
//   the waves' sums are added in order.  Bound by the two erfc per bin and cut: 4000 bins and
//   40000 cuts took 2241 us with a thread per cut, 750 us here.
// * pld_masses_kernel: cell masses of the grid t_j = (j - n + 1) h, j < 2n - 1,
//   as decrements of S between the cuts around each cell (clamped at zero); the
//   mass below the first cut joins the lowest cell, S at the last cut is the atom
//   at +infinity; everything is normalised to total one.
// * pld_fold_kernel: after a linear convolution of two such distributions (an FFT
//   product computed by the caller), negatives are clipped, the centred L cells
//   are kept, mass below them is folded into the lowest cell, mass above joins the
//   +infinity atom (whose mass composes as 1 - (1 - a)(1 - b)), and the finite
//   cells are rescaled so that the total stays one.
// * pld_delta_kernel: delta(eps) = sum over t_j >= eps of q_j (1 - e^(eps - t_j))
//   plus the atom, clipped to [0, 1], for a batch of eps values (one workgroup each).
//
// Every reduction runs within a workgroup in a fixed order, so results are
// deterministic.  Phi is the standard normal CDF, 0.5 erfc(-x / sqrt 2).
#include <algorithm>
#include "device.hpp"
#include "kernels.hpp"

namespace dprc {

constexpr int kPldBlock = 1024;

__device__ __forceinline__ double norm_cdf(double x) { return 0.5 * erfc(-x * 0.70710678118654752440); }

// Sum of the workgroup's `v` (fixed order: lanes within each wave, then waves in order).
__device__ double block_sum(double v, double* red) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if (lane == 0) red[wv] = v;
  __syncthreads();
  double s = 0.0;
  for (int q = 0; q < nw; ++q) s += red[q];
  return s;
}

__global__ __launch_bounds__(kPldBlock) void envelope_bins_kernel(const double* F, int32_t M, double y_min,
                                                                  double y_max, double* ybar, double* w) {
  __shared__ double cmax[kPldBlock];
  __shared__ double red[kPldBlock / 64];
  const int tid = threadIdx.x;
  const int64_t npts = (int64_t)M + 1;
  const int64_t chunk = (npts + kPldBlock - 1) / kPldBlock;
  const int64_t b0 = tid * chunk, b1 = min(npts, b0 + chunk);
  // running maximum: each thread's chunk maximum, then a prefix maximum over the chunks
  double m = -INFINITY;
  for (int64_t j = b0; j < b1; ++j) m = fmax(m, F[j]);
  cmax[tid] = m;
  __syncthreads();
  for (int off = 1; off < kPldBlock; off <<= 1) {   // inclusive prefix maximum (Hillis-Steele)
    const double o = tid >= off ? cmax[tid - off] : -INFINITY;
    __syncthreads();
    cmax[tid] = fmax(cmax[tid], o);
    __syncthreads();
  }
  const double before = tid > 0 ? cmax[tid - 1] : -INFINITY;
  // weights of bins j = b0 .. b1 - 1 (bin j spans points j, j + 1); a chunk's last bin
  // needs the next chunk's first point, which the running maximum through it gives
  double run = before, local = 0.0;
  for (int64_t j = b0; j < b1 && j < M; ++j) {
    run = fmax(run, F[j]);
    const double g0 = fmin(fmax(run, 0.0), 1.0);
    const double g1 = fmin(fmax(fmax(run, F[j + 1]), 0.0), 1.0);
    const double wj = fmax(g1 - g0, 0.0);
    w[j] = wj;
    local += wj;
  }
  const double tot = block_sum(local, red);
  const double step = (y_max - y_min) / (double)M;
  for (int64_t j = b0; j < b1 && j < M; ++j) {
    w[j] = w[j] / tot;
    ybar[j] = y_min + ((double)j + 0.5) * step;
  }
}

constexpr int kSurvWaves = 8;
__global__ __launch_bounds__(64 * kSurvWaves) void pld_survival_kernel(PldArgs a) {
  __shared__ double tab[kSurvWaves][64][3];      // a wave's next 64 bins: 1/mu, mu/2, weight
  __shared__ double sums[kSurvWaves][64][2];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t c = (int64_t)blockIdx.x * 64 + lane;
  const double t = ((double)(c - a.n) + 0.5) * a.h;
  const bool inside = c < 2 * a.n && t > a.t_min;
  const double u = inside && a.p < 1.0 ? t + log(1.0 / a.p - (1.0 - a.p) / a.p * exp(-t)) : t;
  double al = 0.0, beb = 0.0;
  if (a.n_bins == 0) {
    const double mu = 1.0 / a.sigma;
    al = norm_cdf(-u / mu - 0.5 * mu);
    beb = norm_cdf(-u / mu + 0.5 * mu);
  } else if (__syncthreads_or(inside)) {         // (a group of cuts at or below the support does nothing)
    const int32_t per = (a.n_bins + kSurvWaves - 1) / kSurvWaves;
    const int32_t i1 = min(a.n_bins, (wv + 1) * per);
    for (int32_t i0 = wv * per; i0 < i1; i0 += 64) {
      const int32_t i = i0 + lane;
      const double inv = i < i1 ? sqrt(a.ybar[i]) * a.sigma : 1.0;
      tab[wv][lane][0] = inv;
      tab[wv][lane][1] = 0.5 / inv;
      tab[wv][lane][2] = i < i1 ? a.w[i] : 0.0;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const int m = min(64, i1 - i0);
      for (int k = 0; k < m; ++k) {
        const double wi = tab[wv][k][2];
        if (wi == 0.0) continue;                 // the same for the whole wave
        const double z = -u * tab[wv][k][0], hm = tab[wv][k][1];
        al += wi * norm_cdf(z - hm);
        beb += wi * norm_cdf(z + hm);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    sums[wv][lane][0] = al;
    sums[wv][lane][1] = beb;
    __syncthreads();
    if (wv == 0)
      for (int w = 1; w < kSurvWaves; ++w) {
        al += sums[w][lane][0];
        beb += sums[w][lane][1];
      }
  }
  if (wv == 0 && c < 2 * a.n) a.S[c] = inside ? a.p * beb + (1.0 - a.p) * al : 1.0;
}

// Sum over j in [b, e) of f(j) (threads stride by the workgroup, eight values in flight per
// thread).
template <class F>
__device__ __forceinline__ double strided_sum(int64_t b, int64_t e, F&& f) {
  constexpr int U = 8;
  double s = 0.0;
  for (int64_t j0 = b + threadIdx.x; j0 < e; j0 += (int64_t)U * blockDim.x) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t j = j0 + (int64_t)u * blockDim.x;
      v[u] = j < e ? f(j) : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) s += v[u];
  }
  return s;
}

// The cells of one of the gridDim.x equal parts of [0, L).
__device__ __forceinline__ void grid_part(int64_t L, int64_t& b, int64_t& e) {
  const int64_t per = (L + gridDim.x - 1) / gridDim.x;
  b = (int64_t)blockIdx.x * per;
  e = min(L, b + per);
}

// The normalisers below are sums over the whole grid.  Every workgroup of the launch adds
// the same values in the same order (1.3 MB out of L2 for 80000 cells) and writes its own
// part of the cells, which needs no scratch memory and no second launch: 113 us with one
// workgroup of contiguous chunks, 27 us with kPldParts of strided ones.
constexpr int kPldParts = 16;

__global__ __launch_bounds__(kPldBlock) void pld_masses_kernel(PldArgs a) {
  __shared__ double red[kPldBlock / 64];
  const int64_t L = 2 * a.n - 1;
  auto mass = [&](int64_t j) {
    const double qj = fmax(a.S[j] - a.S[j + 1], 0.0);
    return j == 0 ? qj + fmax(1.0 - a.S[0], 0.0) : qj;   // below the first cut
  };
  const double atom = fmax(a.S[2 * a.n - 1], 0.0);  // above the last cut
  const double tot = block_sum(strided_sum(0, L, mass), red) + atom;
  int64_t b, e;
  grid_part(L, b, e);
  for (int64_t j = b + threadIdx.x; j < e; j += blockDim.x) a.q[j] = mass(j) / tot;
  if (blockIdx.x == 0 && threadIdx.x == 0) a.q_inf[0] = atom / tot;
}

__global__ __launch_bounds__(kPldBlock) void pld_fold_kernel(const double* r, int64_t L, const double* ainf,
                                                             const double* binf, double* q, double* q_inf) {
  __shared__ double red[kPldBlock / 64];
  const int64_t n = 2 * L - 1, c = (L - 1) / 2;       // r[j] sits at cell j - c of the kept grid
  auto pos = [&](int64_t j) { return fmax(r[j], 0.0); };
  const double below = block_sum(strided_sum(0, c, pos), red);
  const double kept = block_sum(strided_sum(c, c + L, pos), red);
  const double above = block_sum(strided_sum(c + L, n, pos), red);
  const double inf0 = 1.0 - (1.0 - ainf[0]) * (1.0 - binf[0]);
  const double fin = below + kept + above;
  const double scale = fin > 0.0 ? (1.0 - inf0) / fin : 0.0;
  int64_t b, e;
  grid_part(L, b, e);
  for (int64_t j = b + threadIdx.x; j < e; j += blockDim.x) q[j] = (j == 0 ? pos(c) + below : pos(c + j)) * scale;
  if (blockIdx.x == 0 && threadIdx.x == 0) q_inf[0] = fin > 0.0 ? inf0 + above * scale : inf0;
}

// One workgroup per eps.
__global__ __launch_bounds__(kPldBlock) void pld_delta_kernel(const double* q, int64_t L, double h, const double* q_inf,
                                                              const double* eps, double* delta) {
  __shared__ double red[kPldBlock / 64];
  const double e = eps[blockIdx.x];
  const int64_t c = (L - 1) / 2;
  const double s = strided_sum(0, L, [&](int64_t j) {
    const double t = (double)(j - c) * h;
    return t >= e ? q[j] * (1.0 - exp(e - t)) : 0.0;
  });
  const double tot = block_sum(s, red) + q_inf[0];
  if (threadIdx.x == 0) delta[blockIdx.x] = fmin(fmax(tot, 0.0), 1.0);
}

hipError_t launch_envelope_bins(const double* F, int32_t M, double y_min, double y_max, double* ybar, double* w,
                                hipStream_t st) {
  DPRC_LAUNCH(envelope_bins_kernel, dim3(1), dim3(kPldBlock), 0, st, F, M, y_min, y_max, ybar, w);
  return hipGetLastError();
}

hipError_t launch_pld_step(const PldArgs& a, hipStream_t st) {
  DPRC_LAUNCH(pld_survival_kernel, dim3((unsigned)ceil_div(2 * a.n, 64)), dim3(64 * kSurvWaves), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  DPRC_LAUNCH(pld_masses_kernel, dim3(kPldParts), dim3(kPldBlock), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_pld_fold(const double* r, int64_t L, const double* ainf, const double* binf, double* q,
                           double* q_inf, hipStream_t st) {
  DPRC_LAUNCH(pld_fold_kernel, dim3(kPldParts), dim3(kPldBlock), 0, st, r, L, ainf, binf, q, q_inf);
  return hipGetLastError();
}

hipError_t launch_pld_delta(const double* q, int64_t L, double h, const double* q_inf, const double* eps,
                            int32_t n_eps, double* delta, hipStream_t st) {
  DPRC_LAUNCH(pld_delta_kernel, dim3((unsigned)n_eps), dim3(kPldBlock), 0, st, q, L, h, q_inf, eps, delta);
  return hipGetLastError();
}

}  // namespace dprc
