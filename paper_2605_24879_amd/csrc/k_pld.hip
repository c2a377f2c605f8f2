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
//   A workgroup of eight waves takes 16 cut points; a wave sums its eighth of the bins for
//   all of them (four lanes per cut; the bins' 1/mu and mu/2 are computed once per wave), and
//   the lanes' and waves' sums are added in order.  Bound by fp64 arithmetic, two normal
//   tails per bin and cut: 4000 bins and 40000 cuts took 2241 us with a thread per cut and two
//   erfc per bin, 327 us here (750 with erfc and 64 cuts per workgroup, 590 with the shared
//   exponential; the 20000 cuts above the support then left a third of the CUs idle at the end).
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

// e^(x^2) erfc(x) for x >= 0: (1 + 2x) times it is smooth on [0, inf] in t = (x - 3.75) /
// (x + 3.75) (Shepherd and Laframboise, Math. Comp. 36, 1981); the polynomial interpolates it
// at 25 Chebyshev nodes (computed in 50 digits), relative error below 3e-16 on [0, 50].
__device__ __forceinline__ double erfcx_pos(double x) {
  constexpr double c[25] = {
    1.23751263083782748e+00, -1.40240598585546966e-01, 3.58541548546377487e-03, 8.22767384901451626e-02,
    -1.08803930141717853e-01, 9.23043211603787606e-02, -5.86933985902123659e-02, 2.83622774189406651e-02,
    -9.74657955250424375e-03, 1.75562585300172570e-03, 2.93713634285008114e-04, -2.90154080979527107e-04,
    5.16492113907028545e-05, 2.23842403142244369e-05, -1.14444124391717224e-05, -9.73561901518266272e-07,
    1.75205797016631802e-06, -5.72159725599098732e-08, -2.59106968779665778e-07, 2.32619132766965658e-08,
    3.89654525489859656e-08, -3.74356803363458306e-09, -5.28428697963142026e-09, 3.11031071983916516e-10,
    4.43495907000962802e-10};
  const double a = x + 3.75, b = fma(2.0, x, 1.0), r = 1.0 / (a * b);
  const double t = (x - 3.75) * b * r;
  double v = c[24];
#pragma unroll
  for (int k = 23; k >= 0; --k) v = fma(v, t, c[k]);
  return v * (a * r);
}

// Phi(-w) given e = exp(-w^2 / 2) / 2.
__device__ __forceinline__ double upper_tail(double w, double e) {
  const double q = e * erfcx_pos(fmin(fabs(w) * 0.70710678118654752440, 50.0));
  return w >= 0.0 ? q : 1.0 - q;
}

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
constexpr int kSurvCuts = 16;
constexpr double kFarU = 300.0;    // losses above it take an exponential for each tail
__global__ __launch_bounds__(64 * kSurvWaves) void pld_survival_kernel(PldArgs a) {
  __shared__ double tab[kSurvWaves][64][3];      // a wave's next 64 bins: 1/mu, mu/2, weight
  __shared__ double sums[kSurvWaves][kSurvCuts][2];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, cut = lane % kSurvCuts, g = lane / kSurvCuts;
  const int64_t c = (int64_t)flat_block() * kSurvCuts + cut;
  const double t = ((double)(c - a.n) + 0.5) * a.h;
  const bool inside = c < 2 * a.n && t > a.t_min;
  const double u = inside && a.p < 1.0 ? t + log(1.0 / a.p - (1.0 - a.p) / a.p * exp(-t)) : t;
  // e^u leaves the doubles at u = 709.8, and e1 (below) what they resolve before that
  const bool far = u > kFarU;
  const double eu = far ? 0.0 : exp(u);
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
      // a bin without weight has no part in the sums, whatever its point (padding may hold NaN)
      const double wi = i < i1 ? a.w[i] : 0.0;
      const double inv = wi != 0.0 ? sqrt(a.ybar[i]) * a.sigma : 1.0;
      tab[wv][lane][0] = inv;
      tab[wv][lane][1] = 0.5 / inv;
      tab[wv][lane][2] = wi;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const int m = min(64, i1 - i0);
      for (int k = g; k < m; k += 64 / kSurvCuts) {
        // arguments z + h and z - h with z = u / mu, h = mu / 2: 2 z h = u, so one exponential
        // (and e^u, the same for every bin) serves both tails up to kFarU
        const double wi = tab[wv][k][2], hm = tab[wv][k][1], z = u * tab[wv][k][0], w1 = z + hm, w2 = z - hm;
        const double e1 = 0.5 * exp(-0.5 * w1 * w1);
        double e2 = e1 * eu;
        if (far) e2 = 0.5 * exp(-0.5 * w2 * w2);
        al += wi * upper_tail(w1, e1);
        beb += wi * upper_tail(w2, e2);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
#pragma unroll
    for (int m = kSurvCuts; m < 64; m <<= 1) {
      al += __shfl_xor(al, m, 64);
      beb += __shfl_xor(beb, m, 64);
    }
    if (g == 0) {
      sums[wv][cut][0] = al;
      sums[wv][cut][1] = beb;
    }
    __syncthreads();
    if (wv == 0)
      for (int w = 1; w < kSurvWaves; ++w) {
        al += sums[w][cut][0];
        beb += sums[w][cut][1];
      }
  }
  if (wv == 0 && g == 0 && c < 2 * a.n) a.S[c] = inside ? a.p * beb + (1.0 - a.p) * al : 1.0;
}

// Sum over j in [b, e) of f(j) (threads stride by the workgroup, 16 values in flight per
// thread).
template <class F>
__device__ __forceinline__ double strided_sum(int64_t b, int64_t e, F&& f) {
  constexpr int U = 16;
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

// The masses' normaliser is a sum over the whole grid.  Every workgroup of the launch adds
// the same values in the same order (0.3 MB out of L2 for 40000 cells) and writes its own
// part of the cells, which needs no scratch memory and no second launch: 113 us with one
// workgroup of contiguous chunks, 16 us with kPldParts of strided ones.
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

// The fold reads twice as much as it writes, and one CU streams about 45 GB/s (1.3 MB took
// 28 us that way), so its sums are split over kFoldParts workgroups.  There is no scratch
// memory: the partial sums go to the front of q, a second launch turns every other cell
// out, and a third, of one workgroup, the cells that held them.  Below kFoldWhole cells one
// workgroup does it all (12001 cells: 11.8 us against 13.3, 2001: 8.0 and 13.7; 20001: 15.5
// and 13.6).
constexpr int kFoldParts = 64, kFoldBlock = 256, kFoldHead = 3 * kFoldParts;
constexpr int64_t kFoldWhole = 15000;
static_assert(kFoldWhole > kFoldHead, "the partial sums fit the grid");

struct FoldRange {                                    // r[j] sits at cell j - c of the kept grid
  int64_t n, c;
};
__device__ __forceinline__ FoldRange fold_range(int64_t L) { return {2 * L - 1, (L - 1) / 2}; }

// Sums below, inside and above the kept grid over part b of nb of r, to the whole workgroup.
__device__ __forceinline__ void fold_part(const double* r, int64_t L, int b, int nb, double* red, double (&s)[3]) {
  const FoldRange f = fold_range(L);
  const int64_t per = (f.n + nb - 1) / nb, j0 = b * per, j1 = min(f.n, j0 + per);
  auto pos = [&](int64_t j) { return fmax(r[j], 0.0); };
  s[0] = block_sum(strided_sum(j0, min(j1, f.c), pos), red);
  s[1] = block_sum(strided_sum(max(j0, f.c), min(j1, f.c + L), pos), red);
  s[2] = block_sum(strided_sum(max(j0, f.c + L), j1, pos), red);
}

// Cells [b, e) and, with `atom`, the atom from the three sums.
__device__ __forceinline__ void fold_cells(const double* r, int64_t L, const double* ainf, const double* binf,
                                           const double (&s)[3], int64_t b, int64_t e, bool atom, double* q,
                                           double* q_inf) {
  const FoldRange f = fold_range(L);
  const double inf0 = 1.0 - (1.0 - ainf[0]) * (1.0 - binf[0]);
  const double fin = s[0] + s[1] + s[2];
  const double scale = fin > 0.0 ? (1.0 - inf0) / fin : 0.0;
  for (int64_t j = b + threadIdx.x; j < e; j += blockDim.x) {
    const double v = fmax(r[f.c + j], 0.0);
    q[j] = (j == 0 ? v + s[0] : v) * scale;
  }
  if (!atom) return;
  __syncthreads();                                    // q_inf may be ainf or binf: every wave has read them
  if (threadIdx.x == 0) q_inf[0] = fin > 0.0 ? inf0 + s[2] * scale : inf0;
}

__global__ __launch_bounds__(kFoldBlock) void pld_fold_sums_kernel(const double* r, int64_t L, double* q) {
  __shared__ double red[kFoldBlock / 64];
  double s[3];
  fold_part(r, L, blockIdx.x, kFoldParts, red, s);
  if (threadIdx.x < 3) q[3 * blockIdx.x + threadIdx.x] = s[threadIdx.x];
}

// head = false: the cells from kFoldHead on, one part per workgroup; head = true: those
// before it, after every workgroup of the other launch has read the partial sums there.
__global__ __launch_bounds__(kPldBlock) void pld_fold_kernel(const double* r, int64_t L, const double* ainf,
                                                              const double* binf, double* q, double* q_inf, bool head,
                                                              bool whole) {
  __shared__ double red[kPldBlock / 64];
  __shared__ double part[kFoldHead];
  double s[3] = {0.0, 0.0, 0.0};
  if (whole) {
    fold_part(r, L, 0, 1, red, s);
    fold_cells(r, L, ainf, binf, s, 0, L, true, q, q_inf);
    return;
  }
  for (int k = threadIdx.x; k < kFoldHead; k += blockDim.x) part[k] = q[k];
  __syncthreads();
  for (int b = 0; b < kFoldParts; ++b)                // every thread, in part order
#pragma unroll
    for (int k = 0; k < 3; ++k) s[k] += part[3 * b + k];
  if (head) {
    fold_cells(r, L, ainf, binf, s, 0, kFoldHead, true, q, q_inf);
  } else {
    int64_t b, e;
    grid_part(L - kFoldHead, b, e);
    fold_cells(r, L, ainf, binf, s, kFoldHead + b, kFoldHead + e, false, q, q_inf);
  }
}

// One workgroup per eps.
__global__ __launch_bounds__(kPldBlock) void pld_delta_kernel(const double* q, int64_t L, double h, const double* q_inf,
                                                              const double* eps, double* delta) {
  __shared__ double red[kPldBlock / 64];
  const double e = eps[blockIdx.x];
  const int64_t c = (L - 1) / 2;
  // the cells from two below eps on, in runs of 16 per thread: one exponential per run, the
  // others by the constant ratio between a thread's cells.  The first exponent, at most 3 h,
  // is kept where e^x is a double: beyond that the ratio is 0, and 0 has to follow.
  constexpr int U = 16;
  const double ratio = exp(-(double)blockDim.x * h);
  const double first = floor(e / h) + (double)(c - 2);
  const int64_t j1 = first <= 0.0 ? 0 : (first < (double)L ? (int64_t)first : L);   // eps not a number: no cell
  double s = 0.0;
  for (int64_t j0 = j1 + threadIdx.x; j0 < L; j0 += (int64_t)U * blockDim.x) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = q[min(j0 + (int64_t)u * blockDim.x, L - 1)];
    double ex = exp(fmin(e - (double)(j0 - c) * h, 700.0));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t j = j0 + (int64_t)u * blockDim.x;
      if (j < L && (double)(j - c) * h >= e) s += v[u] * (1.0 - ex);
      ex *= ratio;
    }
  }
  const double tot = block_sum(s, red) + q_inf[0];
  if (threadIdx.x == 0) delta[blockIdx.x] = fmin(fmax(tot, 0.0), 1.0);
}

hipError_t launch_envelope_bins(const double* F, int32_t M, double y_min, double y_max, double* ybar, double* w,
                                hipStream_t st) {
  DPRC_LAUNCH(envelope_bins_kernel, dim3(1), dim3(kPldBlock), 0, st, F, M, y_min, y_max, ybar, w);
  return hipGetLastError();
}

hipError_t launch_pld_step(const PldArgs& a, hipStream_t st) {
  DPRC_LAUNCH(pld_survival_kernel, flat_grid(ceil_div(2 * a.n, kSurvCuts)), dim3(64 * kSurvWaves), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  DPRC_LAUNCH(pld_masses_kernel, dim3(kPldParts), dim3(kPldBlock), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_pld_fold(const double* r, int64_t L, const double* ainf, const double* binf, double* q,
                           double* q_inf, hipStream_t st) {
  const bool whole = L < kFoldWhole;
  if (!whole) {
    DPRC_LAUNCH(pld_fold_sums_kernel, dim3(kFoldParts), dim3(kFoldBlock), 0, st, r, L, q);
    DPRC_LAUNCH(pld_fold_kernel, dim3(kFoldParts), dim3(kFoldBlock), 0, st, r, L, ainf, binf, q, q_inf, false, false);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  DPRC_LAUNCH(pld_fold_kernel, dim3(1), dim3(whole ? kPldBlock : kFoldBlock), 0, st, r, L, ainf, binf, q, q_inf, true,
              whole);
  return hipGetLastError();
}

hipError_t launch_pld_delta(const double* q, int64_t L, double h, const double* q_inf, const double* eps,
                            int32_t n_eps, double* delta, hipStream_t st) {
  // One workgroup per eps: of 1024 threads while a CU has at most two, of 256 where many eps
  // fill the GPU anyway (1000 eps: 17.8 us on 16383 cells, 24.7 on 39999 and 10.4 on one with
  // 1024 threads, 8.3, 15.8 and 7.0 with 256; 64 eps on 400001 cells: 36 and 73).
  DPRC_LAUNCH(pld_delta_kernel, dim3((unsigned)n_eps), dim3(n_eps > 512 ? 256 : kPldBlock), 0, st, q, L, h, q_inf, eps, delta);
  return hipGetLastError();
}

}  // namespace dprc
