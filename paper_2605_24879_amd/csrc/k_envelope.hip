// Envelope CDF of the Hutchinson estimate (privacy analysis, proposition on the
// extremal envelope; appendix algorithms cdf-grid and binary-search-xplus).
//
// MiddleRegionCDF(x): the largest P(S <= x) over the two-level forms
//   S(i, j, lam) = lam/(ik) chi^2(ik) + (1-lam)/(jk) chi^2(jk),
//   i, j >= 1, i + j <= d, lam = l / (2 (n_lambda - 1)), l = 0 .. n_lambda - 1.
// Four lanes per candidate (i, j, l) and point x (fp64).  A candidate's CDF is
// the convolution integral over the first term written in s = sqrt(v) (v the
// chi^2(ik) variable), where the chi density has a bulk of constant width:
//   P(S <= x) = int 2 s f_{ik}(s^2) G(s) ds,  G(s) = P_reg(jk/2, (x - a s^2)/(2b)),
// a = lam/(ik), b = (1-lam)/(jk), by composite Gauss-Legendre (16-node panels;
// nodes, weights and the integration matrix computed on the host).  G is not
// evaluated at the nodes: its derivative is a gamma density (one log, one exp),
// and within a panel G at the nodes is its value at the panel's start plus the
// integral of the polynomial through the derivative's 16 values (the integration
// matrix), so a candidate needs at most one incomplete gamma, at the start of
// its range.  Panels are at most six standard deviations of the second term
// wide.  Bound by fp64 logs and exponentials (short series about the densities' centres,
// log_ratio and exp_neg): 102816 forms (k = 32, d = 64) took 7.1 ms with an incomplete gamma
// per node and take 0.34 ms here (0.61 with one lane per candidate and 0.43 with the math
// library's log and exp).
// Against 200 panels of 32 nodes the errors are rounding, 1e-12 at most up to k d = 2048 and
// 1e-11 at k = 64, d = 1024, where 16 panels without the width rule were off by 1e-5.  P_reg(a, y) is the power series for
// y < a + 1 and Lentz's evaluation of the Legendre continued fraction for the
// complement otherwise (Press et al., Numerical Recipes, incomplete gamma
// function); lam = 0 reduces to one of them.
// Workgroups reduce (value, candidate index) pairs to the largest value with
// the smallest index; a second kernel reduces the workgroup results.
#include <algorithm>
#include "device.hpp"
#include "kernels.hpp"

namespace dprc {

constexpr int kEnvBlock = 256;
// Lanes per candidate: four, so that a few thousand candidates still fill the GPU, unless
// every form is a single incomplete gamma (lam = 0 only), which four lanes would each compute,
// in a kernel with room for the quadrature: 1540 such forms at 60 points took 56 us that way,
// 20 with a lane each and a kernel of their own.
static int env_lanes(int n_lambda) { return n_lambda > 1 ? 4 : 1; }
constexpr int kEnvRedBlock = 256;

// log(x / c) for positive normal x and c, given inv = 1 / c: with the e that puts x / (2^e c)
// in [sqrt(1/2), sqrt(2)), log(x / (2^e c)) = 2 atanh(s), s = (x - 2^e c) / (x + 2^e c) (the
// difference is exact), by its series to s^23 (|s| <= 0.172: the next term is below 1e-18).
__device__ __forceinline__ double log_ratio(double x, double c, double inv) {
  const double q = x * inv;
  int e = __builtin_amdgcn_frexp_exp(q);
  e = __builtin_amdgcn_frexp_mant(q) < 0.70710678118654752440 ? e - 1 : e;
  const double ce = __builtin_amdgcn_ldexp(c, e), f = x - ce, d = x + ce;
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  r = fma(fma(-d, r, 1.0), r, r);
  double s = f * r;
  s = fma(fma(-d, s, f), r, s);
  const double z = s * s;
  double p = 1.0 / 23.0;
#pragma unroll
  for (int k = 21; k >= 3; k -= 2) p = fma(p, z, 1.0 / k);
  const double ed = (double)e, l = fma(2.0 * s, z * p, 2.0 * s);
  return fma(ed, 0x1.62e42fefa39efp-1, fma(ed, 0x1.abc9e3b39803fp-56, l));   // ln 2 in two parts
}

// log Gamma(h) - [(h - 1/2) log h - h + log(2 pi) / 2], by Stirling's series for large h.
__device__ __forceinline__ double stirling_rest(double h) {
  if (h < 16.0) return lgamma(h) - ((h - 0.5) * log(h) - h + 0.91893853320467274178);
  const double r = 1.0 / h, z = r * r;
  return r * (1.0 / 12 - z * (1.0 / 360 - z * (1.0 / 1260 - z * (1.0 / 1680 - z * (1.0 / 1188)))));
}

// e^x for x below 700 (0 where it underflows): x = n ln 2 + r, |r| <= 0.347, Taylor to r^13.
__device__ __forceinline__ double exp_neg(double x) {
  const double n = rint(x * 1.4426950408889634074);
  const double r = fma(-n, 0x1.abc9e3b39803fp-56, fma(-n, 0x1.62e42fefa39efp-1, x));
  constexpr double c[14] = {1.0, 1.0, 1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720, 1.0 / 5040, 1.0 / 40320,
                            1.0 / 362880, 1.0 / 3628800, 1.0 / 39916800, 1.0 / 479001600, 1.0 / 6227020800.0};
  double v = c[13];
#pragma unroll
  for (int k = 12; k >= 0; --k) v = fma(v, r, c[k]);
  return __builtin_amdgcn_ldexp(v, (int)fmax(n, -4000.0));
}

__device__ double gamma_p(double a, double y) {
  if (y <= 0.0) return 0.0;
  const double lpre = -y + a * log(y) - lgamma(a);
  if (y < a + 1.0) {
    double ap = a, term = 1.0 / a, sum = term;
    for (int n = 0; n < 100000; ++n) {
      ap += 1.0;
      term *= y / ap;
      sum += term;
      if (fabs(term) < fabs(sum) * 1e-17) break;
    }
    return fmin(1.0, sum * exp(lpre));
  }
  const double tiny = 1e-300;
  double b = y + 1.0 - a, c = 1.0 / tiny, d = 1.0 / b, h = d;
  for (int i = 1; i < 100000; ++i) {
    const double an = -i * (i - a);
    b += 2.0;
    d = an * d + b;
    if (fabs(d) < tiny) d = tiny;
    c = b + an / c;
    if (fabs(c) < tiny) c = tiny;
    d = 1.0 / d;
    const double del = d * c;
    h *= del;
    if (fabs(del - 1.0) < 1e-16) break;
  }
  return fmax(0.0, 1.0 - exp(lpre) * h);
}

// P((1 - lam)/n2 chi^2(n2) <= x)
__device__ double second_term_cdf(double x, double n2, double lam) {
  return gamma_p(n2 / 2.0, x / (2.0 * ((1.0 - lam) / n2)));
}

// The value is returned to all LANES consecutive lanes of the candidate; lane `part` of
// them takes every LANES-th run of the panels.
template <int LANES>
__device__ double two_level_cdf(double x, int i, int j, double lam, int k, int part, const EnvArgs& g) {
  if (x <= 0.0) return 0.0;
  const double n1 = (double)i * k, n2 = (double)j * k;
  const double b = (1.0 - lam) / n2;
  if (lam == 0.0) return second_term_cdf(x, n2, lam);
  const double a = lam / n1;
  const double smax = sqrt(x / a), c = sqrt(n1);
  // beyond 7.5 of its centre the chi density of 8 or more degrees is below 1e-15
  const double reach = n1 >= 8.0 ? 7.5 : 10.0;
  const double lo = fmax(0.0, c - reach), hi = fmin(smax, c + reach);
  if (hi <= lo) return 0.0;
  // The chi density 2 s f_{n1}(s^2) and the gamma density of n2/2 relative to their centres
  // c = sqrt(n1) and al = n2/2, where Stirling's formula leaves small constants:
  //   log chi   = (n1 - 1) log(s / c) - (s^2 - n1) / 2 - log(pi) / 2 - rest(n1 / 2),
  //   log gamma = (al - 1) log(y / al) - (y - al) - log(2 pi al) / 2 - rest(al)
  // (summing terms of the size of n log n instead would round at 1e-16 of that).
  const double al = n2 / 2.0, inv2b = 1.0 / (2.0 * b), invc = 1.0 / c, inval = 1.0 / al;
  const double lc = -0.57236494292470008707 - stirling_rest(n1 / 2.0);
  const double lg = -0.5 * log(6.28318530717958647693 * al) - stirling_rest(al);
  const double ab = 2.0 * a * inv2b;                         // |dy/ds| = s 2a / (2b)
  // When the range runs to the end of the support (s = sqrt(x/a)) G vanishes
  // there like (sqrt(x/a) - s)^(n2/2); with s = sqrt(x/a) - t^2 the
  // integrand is smooth in t for every n2.
  const bool edge = hi >= smax;
  const double tlo = edge ? 0.0 : lo, thi = edge ? sqrt(smax - lo) : hi;
  // width in t of the second term's density where s is largest
  const double sd = (1.0 - lam) * sqrt(2.0 / n2) / (2.0 * a * hi);
  const double sdt = edge ? sd / (2.0 * sqrt(fmax(smax - fmax(lo, c - 4.0), 0.25 * (smax - lo)))) : sd;
  const int panels = (int)fmin(fmax(ceil((thi - tlo) / (6.0 * sdt)), 16.0), 1024.0);
  const double pw = (thi - tlo) / panels, half = 0.5 * pw;
  // Over this lane's run of panels: the integral of the chi density (dtot), that of the
  // density times the growth of G since the run's start (ptot), and the growth (gtot).
  const int per = (panels + LANES - 1) / LANES;
  double dtot = 0.0, ptot = 0.0, gtot = 0.0;
  for (int pn = part * per; pn < min(panels, (part + 1) * per); ++pn) {
    const double mid = tlo + (pn + 0.5) * pw;
    double D[kEnvNodes], gd[kEnvNodes];          // weighted chi density, dG/dt
#pragma unroll
    for (int q = 0; q < kEnvNodes; ++q) {
      const double t = mid + half * g.gx[q];
      const double s = edge ? smax - t * t : t;
      const double jac = edge ? 2.0 * t : 1.0;
      // x - a s^2 without its cancellation near the end of the support
      const double rest = edge ? a * t * t * (2.0 * smax - t * t) : x - a * s * s;
      const bool ok = s > 0.0 && rest > 0.0;
      const double so = ok ? s : c, y = ok ? rest * inv2b : al;
      const double dens = jac * exp_neg(lc + ((n1 - 1.0) * log_ratio(so, c, invc) - 0.5 * (so - c) * (so + c)));
      const double der = (edge ? jac : -1.0) * ab * so *
                         exp_neg(lg + ((al - 1.0) * log_ratio(y, al, inval) - (y - al)));
      D[q] = ok ? g.gw[q] * dens : 0.0;
      gd[q] = ok ? der : 0.0;
    }
    double ps = 0.0, dsum = 0.0, gsum = 0.0;
#pragma unroll
    for (int q = 0; q < kEnvNodes; ++q) {
      double gq = 0.0;
#pragma unroll
      for (int e = 0; e < kEnvNodes; ++e) gq = fma(g.gi[q][e], gd[e], gq);
      ps = fma(D[q], gq, ps);
      dsum += D[q];
      gsum = fma(g.gw[q], gd[q], gsum);
    }
    ptot += half * (gtot * dsum + half * ps);
    dtot += half * dsum;
    gtot += half * gsum;
  }
  double G0 = edge ? 0.0 : gamma_p(al, (x - a * lo * lo) * inv2b);
  double sum = 0.0;
  const int lane0 = (threadIdx.x & 63) - part;
#pragma unroll
  for (int r = 0; r < LANES; ++r) {                // the runs in order, each from G at its start
    sum += G0 * __shfl(dtot, lane0 + r, 64) + __shfl(ptot, lane0 + r, 64);
    G0 += __shfl(gtot, lane0 + r, 64);
  }
  return fmin(fmax(sum, 0.0), 1.0);
}

// candidate c -> (i, j, l): pairs in (i, then j) order, lam index fastest
__device__ void candidate(int64_t c, int d, int nl, int& i, int& j, int& l) {
  l = (int)(c % nl);
  int64_t pr = c / nl;
  // row i (1-based) holds d - i pairs; offset(i) = (i-1) d - (i-1) i / 2
  int lo = 1, hi = d - 1;
  while (lo < hi) {
    const int m = (lo + hi + 1) / 2;
    const int64_t off = (int64_t)(m - 1) * d - (int64_t)(m - 1) * m / 2;
    if (off <= pr) lo = m;
    else hi = m - 1;
  }
  i = lo;
  j = 1 + (int)(pr - ((int64_t)(i - 1) * d - (int64_t)(i - 1) * i / 2));
}

__device__ __forceinline__ void better(double v, int64_t c, double& bv, int64_t& bc) {
  if (v > bv || (v == bv && c < bc)) { bv = v; bc = c; }
}

template <int LANES>
__global__ __launch_bounds__(kEnvBlock) __attribute__((amdgpu_waves_per_eu(2))) void env_middle_kernel(EnvArgs a) {
  __shared__ double sv[kEnvBlock];
  __shared__ int64_t sc[kEnvBlock];
  const int xi = blockIdx.y;
  const double x = a.x[xi];
  double bv = -1.0;
  int64_t bc = INT64_MAX;
  // (the lanes of a candidate share c, so they leave the loop and return early together)
  for (int64_t c = (int64_t)blockIdx.x * (kEnvBlock / LANES) + threadIdx.x / LANES; c < a.ncand;
       c += (int64_t)gridDim.x * (kEnvBlock / LANES)) {
    int i, j, l;
    candidate(c, a.d, a.n_lambda, i, j, l);
    const double lam = a.n_lambda > 1 ? 0.5 * l / (a.n_lambda - 1) : 0.0;
    double v;
    if constexpr (LANES > 1) v = two_level_cdf<LANES>(x, i, j, lam, a.k, threadIdx.x % LANES, a);
    else v = second_term_cdf(x, (double)j * a.k, lam);
    better(v, c, bv, bc);
  }
  sv[threadIdx.x] = bv;
  sc[threadIdx.x] = bc;
  __syncthreads();
  for (int off = kEnvBlock / 2; off > 0; off >>= 1) {
    if (threadIdx.x < off) {
      double v = sv[threadIdx.x];
      int64_t c = sc[threadIdx.x];
      better(sv[threadIdx.x + off], sc[threadIdx.x + off], v, c);
      sv[threadIdx.x] = v;
      sc[threadIdx.x] = c;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    a.part_v[(int64_t)xi * gridDim.x + blockIdx.x] = sv[0];
    a.part_c[(int64_t)xi * gridDim.x + blockIdx.x] = sc[0];
  }
}

__global__ __launch_bounds__(kEnvRedBlock) void env_reduce_kernel(EnvArgs a, int nblk) {
  __shared__ double sv[kEnvRedBlock / 64];
  __shared__ int64_t sc[kEnvRedBlock / 64];
  const int xi = blockIdx.x, tid = threadIdx.x;
  double bv = -1.0;
  int64_t bc = INT64_MAX;
  for (int b = tid; b < nblk; b += kEnvRedBlock)
    better(a.part_v[(int64_t)xi * nblk + b], a.part_c[(int64_t)xi * nblk + b], bv, bc);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) better(__shfl_xor(bv, off, 64), __shfl_xor(bc, off, 64), bv, bc);
  if ((tid & 63) == 0) {
    sv[tid >> 6] = bv;
    sc[tid >> 6] = bc;
  }
  __syncthreads();
  if (tid != 0) return;
  for (int w = 1; w < kEnvRedBlock / 64; ++w) better(sv[w], sc[w], bv, bc);
  a.best[xi] = bv;
  if (a.arg) {
    int i, j, l;
    candidate(bc, a.d, a.n_lambda, i, j, l);
    a.arg[3 * xi] = i;
    a.arg[3 * xi + 1] = j;
    a.arg[3 * xi + 2] = l;
  }
}

__global__ void chi2_cdf_kernel(const double* x, int64_t n, double dof, double scale, double* out) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    out[e] = gamma_p(dof / 2.0, x[e] * scale / 2.0);
}

hipError_t launch_chi2_cdf(const double* x, int64_t n, double dof, double scale, double* out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)std::min<int64_t>(4096, ceil_div(n, 256));
  DPRC_LAUNCH(chi2_cdf_kernel, dim3(blocks), dim3(256), 0, st, x, n, dof, scale, out);
  return hipGetLastError();
}

int env_blocks(int64_t ncand, int n_lambda) {
  return (int)std::min<int64_t>(2048, ceil_div(ncand, kEnvBlock / env_lanes(n_lambda)));
}

hipError_t launch_env_middle(const EnvArgs& a, hipStream_t st) {
  const int nblk = env_blocks(a.ncand, a.n_lambda);
  const dim3 grid((unsigned)nblk, (unsigned)a.nx);
  if (env_lanes(a.n_lambda) == 4) DPRC_LAUNCH(env_middle_kernel<4>, grid, dim3(kEnvBlock), 0, st, a);
  else DPRC_LAUNCH(env_middle_kernel<1>, grid, dim3(kEnvBlock), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  DPRC_LAUNCH(env_reduce_kernel, dim3((unsigned)a.nx), dim3(kEnvRedBlock), 0, st, a, nblk);
  return hipGetLastError();
}

}  // namespace dprc
