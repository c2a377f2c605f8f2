// Hutch++ pieces that are not token streams (Algorithm 2, Hutch++ branch):
//
//  * Q = orthonormal basis of the sketch O S (m x s per sample) by a tall-skinny
//    Householder QR as a tree: one wavefront factors a block of 128 rows held in
//    registers (two rows per lane, fp64), the s x s R factors of the blocks are
//    stacked and factored the same way at the next level, until one block is
//    left.  The expansion runs back down the tree: each block starts from its s
//    rows of the level above's Q (the identity at the top) and applies its own
//    reflectors.  One launch takes the same step of up to eight layers' trees
//    (each block finds its layer from its block index), so the latency-bound tree
//    costs a few launches per call rather than a few per layer.  Householder keeps Q orthonormal when O S is rank deficient (a
//    Gram/Cholesky QR breaks down there).  Dot products over a block's rows are
//    summed across the wave through LDS in a fixed order, so the result does not
//    depend on scheduling.
//  * While it holds its rows of Q, a level-1 block also forms its share of
//    C = Q^T P (P the residual probes, regenerated from Philox).
//  * The finalize step V = W_P - U C and the sums ||U||^2, ||V||^2 run
//    row-parallel; a last kernel adds the row chunks in a fixed order:
//    estimate = ||U||^2 + ||V||^2 / r.
#include <algorithm>
#include "device.hpp"
#include "kernels.hpp"

namespace dprc {

constexpr int kQrThreads = 256;   // finalize kernels
constexpr int kRedLd = 65;        // padded row of the per-column lane sums

__device__ __forceinline__ double qr_block_sum(double v, double* sh) {
  const int tid = threadIdx.x;
  v = wave_sum(v);
  __syncthreads();
  if ((tid & 63) == 0) sh[tid >> 6] = v;
  __syncthreads();
  return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// Orders a wave's LDS accesses around a hand-off between its lanes (LDS
// operations of one wave execute in issue order; this keeps the compiler from
// moving them across).
__device__ __forceinline__ void qr_wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ double readlane_f64(double v, int l) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// x[l] + x[l ^ 16] (R = 16) or x[l] + x[l ^ 32] (R = 32) with the lane swaps of
// gfx950: the swap returns the pair's two values in the same order on both lanes
// (lane with the bit clear first), so both lanes form the same sum.
template <int R>
__device__ __forceinline__ double add_across(double x) {
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  const uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
  uint32_t l0, l1, h0, h1;
  if constexpr (R == 16) {
    const auto pl = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto ph = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    l0 = pl[0]; l1 = pl[1]; h0 = ph[0]; h1 = ph[1];
  } else {
    const auto pl = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto ph = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    l0 = pl[0]; l1 = pl[1]; h0 = ph[0]; h1 = ph[1];
  }
  return __longlong_as_double((long long)(((uint64_t)h0 << 32) | l0)) +
         __longlong_as_double((long long)(((uint64_t)h1 << 32) | l1));
}

// v[c] <- sum over the 64 lanes of v[c], for c >= c_lo (c_lo a constant after
// unrolling).  Lane sums go to LDS column by column; lane (c, g) adds the g-th
// run of SP of them, and shuffles over the run bits finish the sum.
template <int SP>
__device__ __forceinline__ void wave_vec_sum(double (&v)[SP], int c_lo, double* red, double* tot) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int c = 0; c < SP; ++c)
    if (c >= c_lo) red[c * kRedLd + lane] = v[c];
  qr_wave_fence();
  const int c = lane % SP, g = lane / SP;
  double x = 0.0;
  if (c >= c_lo) {
    double t[SP];                                 // all reads in flight before the adds
#pragma unroll
    for (int q = 0; q < SP; ++q) t[q] = red[c * kRedLd + g * SP + q];
#pragma unroll
    for (int w = SP / 2; w >= 1; w >>= 1)        // pairwise tree
#pragma unroll
      for (int q = 0; q < w; ++q) t[q] += t[q + w];
    x = t[0];
  }
#pragma unroll
  for (int e = 0; e < 6; ++e) {
    const int m = SP << e;
    if (m == 16) x = add_across<16>(x);
    else if (m == 32) x = add_across<32>(x);
    else if (m < 64) x += __shfl_xor(x, m, 64);
  }
  if (g == 0) tot[c] = x;
  qr_wave_fence();
#pragma unroll
  for (int q = 0; q < SP; ++q)
    if (q >= c_lo) v[q] = tot[q];
  qr_wave_fence();
}

// The job of this block (jobs start at increasing blk0) and its (block, sample).
__device__ __forceinline__ int qr_job_index(const QrBatch& bt) {
  int jb = 0;
#pragma unroll
  for (int q = 1; q < kQrMaxJobs; ++q) jb += (q < bt.njobs && flat_block() >= bt.job[q].blk0) ? 1 : 0;
  return jb;
}

// f(QInt<I>{}) for I = B, B + 1, ..., E - 1.
template <int V>
struct QInt {
  static constexpr int value = V;
};
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(QInt<B>{});
    static_for<B + 1, E>(f);
  }
}

// ---- factor one 128-row block of a level ----------------------------------------------------------
// Lane l holds rows l and l + 64 of the block.  Step k works on column k: v_k = x_k -
// alpha_k e_k over rows >= k, tau_k = 2 / |v_k|^2 (0: identity reflector for a zero column),
// alpha_k = R_kk; the dot products v_k . A_c come from one pass with the norm: x_k . A_c -
// alpha_k A_kc.  v_k stays in column k (rows >= k) and row k of R in lane k's row (columns
// > k, with alpha_k kept apart) until the block is done.  The steps are unrolled: each works
// on the columns it still has, with constant register indices (a loop that moved the
// remaining columns down one register per step, and kept them all, took 17 to 20 us per level
// at 16 columns, this takes 12 to 15).
template <int SP>
__global__ __launch_bounds__(64) void qr_factor_kernel(QrBatch bt) {
  __shared__ double red[SP * kRedLd];
  __shared__ double tot[SP];
  if (blockIdx.y > 0 && flat_block() >= bt.blocks) return;     // (the first row is full)
  const QrJob& a = bt.job[qr_job_index(bt)];
  const int level = a.level;
  const int rel = flat_block() - a.blk0;
  const int b = rel % a.L.nblk, i = rel / a.L.nblk, lane = threadIdx.x;
  const int s = a.s;
  const QrLevel L = a.L;
  // all loads are issued before the first use: masked entries read a valid address
  // and are replaced by zero
  double A[2][SP];
  if (level == 0) {
    const float* os = a.OS + (int64_t)i * a.os_ss;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int row = b * kQrRows + lane + 64 * u;
#pragma unroll
      for (int c = 0; c < SP; ++c) {
        const bool ok = c < s && row < L.rows;
        const float x = os[ok ? (int64_t)c * a.os_ld + row : 0];
        A[u][c] = ok ? (double)x : 0.0;
      }
    }
  } else {
    const double* ms = L.M + (int64_t)i * s * L.rows;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int row = b * kQrRows + lane + 64 * u;
#pragma unroll
      for (int c = 0; c < SP; ++c) {
        const bool ok = c < s && row < L.rows;
        const double x = ms[ok ? (int64_t)c * L.rows + row : 0];
        A[u][c] = ok ? x : 0.0;
      }
    }
  }
  double* V = L.V + ((int64_t)i * L.nblk + b) * s * kQrRows;
  double* tb = L.tau + ((int64_t)i * L.nblk + b) * s;
  const bool has_next = level + 1 < a.nlev;
  const QrLevel N = has_next ? a.X : a.L;
  double diag = 0.0, tau = 0.0;                     // lane k: alpha_k, tau_k
  static_for<0, SP>([&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value;
    if (k < s) {                                    // uniform
      const double x0k = lane >= k ? A[0][k] : 0.0;
      double pv[SP];
#pragma unroll
      for (int c = k; c < SP; ++c) pv[c] = x0k * A[0][c] + A[1][k] * A[1][c];
      wave_vec_sum<SP>(pv, k, red, tot);
      const double nrm2 = pv[k];
      if (nrm2 > 0.0) {                             // uniform; a zero column keeps the identity reflector
        const double x0 = readlane_f64(A[0][k], k);
        const double al = -copysign(sqrt(nrm2), x0);
        const double v0 = x0 - al;
        const double vn2 = nrm2 - x0 * x0 + v0 * v0;
        const double t = vn2 > 0.0 ? 2.0 / vn2 : 0.0;
        const double tv0 = lane >= k ? t * (lane == k ? v0 : A[0][k]) : 0.0, tv1 = t * A[1][k];
#pragma unroll
        for (int c = k + 1; c < SP; ++c) {
          const double d = pv[c] - al * readlane_f64(A[0][c], k);
          A[0][c] -= tv0 * d;
          A[1][c] -= tv1 * d;
        }
        if (lane == k) {
          A[0][k] = v0;
          diag = al;
          tau = t;
        }
      }
    }
  });
  // V (zero above the diagonal), tau, and the rows of R into rows b*s + q of the next level's
  // input (zero left of the diagonal)
#pragma unroll
  for (int k = 0; k < SP; ++k) {
    if (k < s) {
      V[(int64_t)k * kQrRows + lane] = lane >= k ? A[0][k] : 0.0;
      V[(int64_t)k * kQrRows + lane + 64] = A[1][k];
    }
  }
  if (lane < s) tb[lane] = tau;
  if (has_next && lane < s) {
    double* nm = N.M + (int64_t)i * s * N.rows + (int64_t)b * s + lane;
#pragma unroll
    for (int c = 0; c < SP; ++c)
      if (c < s) nm[(int64_t)c * N.rows] = c > lane ? A[0][c] : (c == lane ? diag : 0.0);
  }
}

// ---- expand one block: W = H_0 ... H_{s-1} [Q_up rows; 0]; level 0 writes Q and C_b = Q_b^T P_b ----
// Wave 0 applies the reflectors (unrolled, as in the factorization).  At level 0 the other
// waves draw the residual probes meanwhile, and all four then form C_b on the fp64 matrix
// cores (16x16x4 MFMA: A[c][j] from the block's Q in LDS, B[j][q] = +-1 from the probe bits;
// D register e of lane l is row 4 e + l / 16, column l % 16).  One wave adding 128 signed rows
// per entry took 37 of the 49 us of a level-0 launch.  Four waves a workgroup while the CUs
// hold them all at once (four, two or one each by registers); beyond that the idle waves'
// registers keep others out, and a workgroup is one wave: 29260 blocks of 16 columns took
// 1177 us with a wave adding signed rows, 1954 with four waves each, 960 with one.
typedef double f64x4_t __attribute__((ext_vector_type(4)));
template <int SP, int NT>
__global__ __launch_bounds__(NT) void qr_expand_kernel(QrBatch bt) {
  __shared__ double red[SP * kRedLd];
  __shared__ double tot[SP];
  constexpr int SR = SP < 16 ? 16 : SP;           // rows of Q in LDS, whole blocks of 16
  constexpr int QLd = kQrRows + 1;
  __shared__ double qs[SR * QLd];
  __shared__ uint32_t zw[256 * 4];
  if (blockIdx.y > 0 && flat_block() >= bt.blocks) return;     // (the first row is full)
  const QrJob& a = bt.job[qr_job_index(bt)];
  const int level = a.level;
  const int rel = flat_block() - a.blk0;
  const int b = rel % a.L.nblk, i = rel / a.L.nblk, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int s = a.s;
  const QrLevel L = a.L;
  if (wv == 0) {
    const bool top = level + 1 == a.nlev;
    const QrLevel U = top ? a.L : a.X;
    // all loads are issued before the first use (masked entries read a valid address)
    double W[2][SP], Vr[2][SP];
    const double* uq = U.Q + (int64_t)i * s * U.rows + (int64_t)b * s;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int j = lane + 64 * u;
#pragma unroll
      for (int c = 0; c < SP; ++c) {
        const bool ok = c < s && j < s;
        double w = 0.0;
        if (top) w = ok && j == c ? 1.0 : 0.0;
        else {
          const double x = uq[ok ? (int64_t)c * U.rows + j : 0];
          w = ok ? x : 0.0;
        }
        W[u][c] = w;
      }
    }
    const double* Vb = L.V + ((int64_t)i * L.nblk + b) * s * kQrRows;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int k = 0; k < SP; ++k) Vr[u][k] = Vb[k < s ? (int64_t)k * kQrRows + lane + 64 * u : 0];
    const double* tb = L.tau + ((int64_t)i * L.nblk + b) * s;
    static_for<0, SP>([&](auto ec) __attribute__((always_inline)) {
      constexpr int k = SP - 1 - decltype(ec)::value;      // reflectors in reverse order
      if (k < s) {                                 // uniform
        const double t = tb[k];
        if (t != 0.0) {
          double pv[SP];
#pragma unroll
          for (int c = 0; c < SP; ++c) pv[c] = Vr[0][k] * W[0][c] + Vr[1][k] * W[1][c];
          wave_vec_sum<SP>(pv, 0, red, tot);
          const double t0 = t * Vr[0][k], t1 = t * Vr[1][k];
#pragma unroll
          for (int c = 0; c < SP; ++c) {
            W[0][c] -= t0 * pv[c];
            W[1][c] -= t1 * pv[c];
          }
        }
      }
    });
    if (level > 0) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int row = b * kQrRows + lane + 64 * u;
        if (row < L.rows) {
#pragma unroll
          for (int c = 0; c < SP; ++c)
            if (c < s) L.Q[((int64_t)i * s + c) * L.rows + row] = W[u][c];
        }
      }
    } else {
      // rows of Q (rows >= m are zero: their reflector entries are zero)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int64_t row = (int64_t)b * kQrRows + lane + 64 * u;
#pragma unroll
        for (int c = 0; c < SR; ++c) {
          const double q = c < SP && c < s && row < a.m ? W[u][c < SP ? c : 0] : 0.0;
          qs[c * QLd + lane + 64 * u] = q;
          if (c < s) {
            if (a.Q && row < a.m) a.Q[(int64_t)i * a.q_ss + (int64_t)c * a.q_ld + row] = (float)q;
            if (a.Qhi && row < a.qh_ld) {
              uint32_t h, l;
              split_bf16((float)q, h, l);
              a.Qhi[(int64_t)i * a.qh_ss + (int64_t)c * a.qh_ld + row] = (uint16_t)h;
              a.Qlo[(int64_t)i * a.qh_ss + (int64_t)c * a.qh_ld + row] = (uint16_t)l;
            }
          }
        }
      }
    }
  }
  if (level == 0 && (NT == 64 || wv > 0)) {
    // probe words of rows b*128 .. b*128+127 (one Philox block per column)
    for (int cc = (int)threadIdx.x - (NT > 64 ? 64 : 0); cc < a.r; cc += NT > 64 ? NT - 64 : 64) {
      const u32x4 v = rademacher_block(a.key0, a.key1, a.layer, kStreamProbe, (uint32_t)b, (uint32_t)cc);
      zw[cc * 4 + 0] = v.x; zw[cc * 4 + 1] = v.y; zw[cc * 4 + 2] = v.z; zw[cc * 4 + 3] = v.w;
    }
  }
  if (level > 0) return;
  __syncthreads();
  // C_b[c][q] = sum_j Q[j][c] z(j, q): blocks of 16 x 16 entries dealt to the waves
  double* cp = a.Cpart + ((int64_t)i * L.nblk + b) * s * a.r;
  const int g = lane >> 4, l16 = lane & 15;
  const int nq = (a.r + 15) / 16, nblocks = (s + 15) / 16 * nq;
  for (int e = wv; e < nblocks; e += NT / 64) {
    const int c0 = 16 * (e / nq), q0 = 16 * (e % nq);
    const double* qa = qs + (c0 + l16) * QLd + g;
    const uint32_t* zq = zw + 4 * min(q0 + l16, a.r - 1);
    f64x4_t acc = {0.0, 0.0, 0.0, 0.0};
    for (int w = 0; w < 4; ++w) {
      const uint32_t bits = zq[w] >> g;
#pragma unroll
      for (int j4 = 0; j4 < 8; ++j4) {
        const double z = (bits >> (4 * j4)) & 1u ? -1.0 : 1.0;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[32 * w + 4 * j4], z, acc, 0, 0, 0);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + 4 * u + g, q = q0 + l16;
      if (c < s && q < a.r) cp[c * a.r + q] = acc[u];
    }
  }
}

int32_t qr_levels(int64_t m, int s, int32_t rows[kQrMaxLevels], int32_t nblk[kQrMaxLevels], int64_t* dbl) {
  int32_t n = 0;
  int64_t r = m, total = 0;
  while (n < kQrMaxLevels) {
    rows[n] = (int32_t)r;
    nblk[n] = (int32_t)ceil_div(r, kQrRows);
    total += (int64_t)nblk[n] * s * kQrRows + (int64_t)nblk[n] * s;   // V, tau
    if (n > 0) total += 2 * r * s;                                     // M, Q
    ++n;
    if (nblk[n - 1] == 1) break;
    r = (int64_t)nblk[n - 1] * s;
  }
  if (nblk[n - 1] != 1) return 0;
  if (dbl) *dbl = total;
  return n;
}

static bool qr_batch_ok(const QrBatch& bt) {
  return bt.s >= 1 && bt.s <= 32 && bt.r <= 256 && bt.njobs >= 1 && bt.njobs <= kQrMaxJobs && bt.blocks >= 1;
}

template <int NT>
static hipError_t launch_qr_expand_t(const QrBatch& bt, hipStream_t st) {
  const dim3 grid = flat_grid(bt.blocks), blk(NT);
  if (bt.s <= 8) DPRC_LAUNCH((qr_expand_kernel<8, NT>), grid, blk, 0, st, bt);
  else if (bt.s <= 16) DPRC_LAUNCH((qr_expand_kernel<16, NT>), grid, blk, 0, st, bt);
  else DPRC_LAUNCH((qr_expand_kernel<32, NT>), grid, blk, 0, st, bt);
  return hipGetLastError();
}

hipError_t launch_qr_factor(const QrBatch& bt, hipStream_t st) {
  if (!qr_batch_ok(bt)) return hipErrorInvalidValue;
  const dim3 grid = flat_grid(bt.blocks), blk(64);
  if (bt.s <= 8) DPRC_LAUNCH(qr_factor_kernel<8>, grid, blk, 0, st, bt);
  else if (bt.s <= 16) DPRC_LAUNCH(qr_factor_kernel<16>, grid, blk, 0, st, bt);
  else DPRC_LAUNCH(qr_factor_kernel<32>, grid, blk, 0, st, bt);
  return hipGetLastError();
}

hipError_t launch_qr_expand(const QrBatch& bt, hipStream_t st) {
  if (!qr_batch_ok(bt)) return hipErrorInvalidValue;
  return bt.blocks <= (bt.s <= 8 ? 1024 : (bt.s <= 16 ? 512 : 256)) ? launch_qr_expand_t<256>(bt, st)
                                                                   : launch_qr_expand_t<64>(bt, st);
}

// ---- finalize -----------------------------------------------------------------------------------------
// A workgroup takes 32 rows j of U | W_P; its threads are (row, column group): group
// g handles the residual columns q = g, g + 8, ..., so a wave reads whole 128-byte
// runs of a column and every row's residuals advance in parallel.
constexpr int kFinRows = 32;                 // rows per workgroup
constexpr int kFinGroups = kQrThreads / kFinRows;

// C = sum of the block partials C_b, in block order (one thread per entry).
__device__ __forceinline__ void hpp_csum_block(const FinalArgs& a, int bx, int i) {
  const int sr = a.s * a.r;
  const int e = bx * kQrThreads + threadIdx.x;
  if (e >= sr) return;
  const double* cp = a.Cpart + (int64_t)i * a.nblk * sr + e;
  double v = 0.0;
  int b = 0;
  for (; b + 8 <= a.nblk; b += 8) {              // eight loads in flight, added in block order
    double x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = cp[(int64_t)(b + u) * sr];
#pragma unroll
    for (int u = 0; u < 8; ++u) v += x[u];
  }
  for (; b < a.nblk; ++b) v += cp[(int64_t)b * sr];
  a.C[(int64_t)i * sr + e] = v;
}
__global__ __launch_bounds__(kQrThreads) void hpp_csum_kernel(FinalArgs a) { hpp_csum_block(a, blockIdx.x, blockIdx.y); }

// Rows of one chunk: ||U_j||^2 and ||W_P,j - U_j C||^2 summed over the chunk.
template <int SP>
__device__ __forceinline__ void hpp_rows_block(const FinalArgs& a, int ch, int i) {
  extern __shared__ __attribute__((aligned(16))) float fs[];
  __shared__ double sh[4];
  const int tid = threadIdx.x;
  const int s = a.s, r = a.r;
  float* C = fs;                           // [s][r]
  for (int e = tid; e < s * r; e += kQrThreads) C[e] = (float)a.C[(int64_t)i * s * r + e];
  __syncthreads();
  const int grp = tid / kFinRows;
  const int64_t j = (int64_t)ch * kFinRows + (tid % kFinRows);
  double su = 0.0, sv = 0.0;
  if (j < a.n) {
    const float* uw = a.UW + (int64_t)i * a.uw_ss + j;
    double u[SP];                                  // row j of U
#pragma unroll
    for (int c = 0; c < SP; ++c) {
      const float x = uw[(int64_t)(c < s ? c : 0) * a.uw_ld];
      u[c] = c < s ? (double)x : 0.0;
      if (grp == 0) su += u[c] * u[c];
    }
    // residual columns of this group, four at a time: their loads are in flight together
    for (int q0 = grp; q0 < r; q0 += 4 * kFinGroups) {
      float w[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int q = q0 + t * kFinGroups;
        w[t] = uw[(int64_t)(s + (q < r ? q : 0)) * a.uw_ld];
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int q = q0 + t * kFinGroups;
        if (q < r) {
          double v = (double)w[t];
#pragma unroll
          for (int c = 0; c < SP; ++c)
            if (c < s) v -= u[c] * (double)C[c * r + q];
          sv += v * v;
        }
      }
    }
  }
  su = qr_block_sum(su, sh);
  sv = qr_block_sum(sv, sh);
  if (tid == 0) {
    a.Fpart[((int64_t)i * a.nchunk + ch) * 2] = su;
    a.Fpart[((int64_t)i * a.nchunk + ch) * 2 + 1] = sv;
  }
}
template <int SP>
__global__ __launch_bounds__(kQrThreads) void hpp_rows_kernel(FinalArgs a) { hpp_rows_block<SP>(a, blockIdx.x, blockIdx.y); }

// The finalize of several layers in one launch per step: block (x, sample) of job j at
// blk0[j] + sample * (x blocks of the job) + x.  The per-sample sum walks the jobs in
// order, so n2 adds the layers' estimates in layer order.
__device__ __forceinline__ int fin_job_index(const FinalBatch& bt) {
  int jb = 0;
#pragma unroll
  for (int q = 1; q < kFinMaxJobs; ++q) jb += (q < bt.njobs && (int)blockIdx.x >= bt.blk0[q]) ? 1 : 0;
  return jb;
}
__global__ __launch_bounds__(kQrThreads) void hpp_csum_batch_kernel(FinalBatch bt) {
  const int jb = fin_job_index(bt);
  const FinalArgs& a = bt.job[jb];
  const int nx = (a.s * a.r + kQrThreads - 1) / kQrThreads;
  const int rel = (int)blockIdx.x - bt.blk0[jb];
  hpp_csum_block(a, rel % nx, rel / nx);
}
template <int SP>
__global__ __launch_bounds__(kQrThreads) void hpp_rows_batch_kernel(FinalBatch bt) {
  const int jb = fin_job_index(bt);
  const FinalArgs& a = bt.job[jb];
  const int rel = (int)blockIdx.x - bt.blk0[jb];
  hpp_rows_block<SP>(a, rel % a.nchunk, rel / a.nchunk);
}

__device__ __forceinline__ void hpp_sum_block(const FinalArgs& a, int i) {
  __shared__ double sh[4];
  double su = 0.0, sv = 0.0;
  for (int c = threadIdx.x; c < a.nchunk; c += kQrThreads) {
    su += a.Fpart[((int64_t)i * a.nchunk + c) * 2];
    sv += a.Fpart[((int64_t)i * a.nchunk + c) * 2 + 1];
  }
  su = qr_block_sum(su, sh);
  sv = qr_block_sum(sv, sh);
  if (threadIdx.x == 0) {
    const float est = (float)(su + sv / (double)a.r);
    a.n2[i] = (a.accumulate ? a.n2[i] : 0.f) + est;
    if (a.n2_layer) a.n2_layer[i] = est;
  }
}
__global__ __launch_bounds__(kQrThreads) void hpp_sum_kernel(FinalArgs a) { hpp_sum_block(a, blockIdx.x); }
__global__ __launch_bounds__(kQrThreads) void hpp_sum_batch_kernel(FinalBatch bt) {
  for (int j = 0; j < bt.njobs; ++j) {               // layer order; each job adds to n2 after the last
    hpp_sum_block(bt.job[j], blockIdx.x);
    __syncthreads();
  }
}

hipError_t launch_hpp_rows(const FinalArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)a.nchunk, (unsigned)a.B);
  const size_t lds = (size_t)a.s * a.r * 4;
  if (a.s <= 8) DPRC_LAUNCH(hpp_rows_kernel<8>, grid, dim3(kQrThreads), lds, st, a);
  else if (a.s <= 16) DPRC_LAUNCH(hpp_rows_kernel<16>, grid, dim3(kQrThreads), lds, st, a);
  else DPRC_LAUNCH(hpp_rows_kernel<32>, grid, dim3(kQrThreads), lds, st, a);
  return hipGetLastError();
}

hipError_t launch_hpp_csum(const FinalArgs& a, hipStream_t st) {
  DPRC_LAUNCH(hpp_csum_kernel, dim3((unsigned)ceil_div((int64_t)a.s * a.r, kQrThreads), (unsigned)a.B),
              dim3(kQrThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_hpp_sum(const FinalArgs& a, hipStream_t st) {
  DPRC_LAUNCH(hpp_sum_kernel, dim3((unsigned)a.B), dim3(kQrThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_hpp_csum_batch(const FinalBatch& bt, hipStream_t st) {
  if (bt.njobs < 1 || bt.njobs > kFinMaxJobs) return hipErrorInvalidValue;
  FinalBatch b = bt;
  int blocks = 0;
  for (int j = 0; j < b.njobs; ++j) {
    b.blk0[j] = blocks;
    blocks += (int)ceil_div((int64_t)b.job[j].s * b.job[j].r, kQrThreads) * b.job[j].B;
  }
  DPRC_LAUNCH(hpp_csum_batch_kernel, dim3((unsigned)blocks), dim3(kQrThreads), 0, st, b);
  return hipGetLastError();
}

hipError_t launch_hpp_rows_batch(const FinalBatch& bt, hipStream_t st) {
  if (bt.njobs < 1 || bt.njobs > kFinMaxJobs) return hipErrorInvalidValue;
  FinalBatch b = bt;
  int blocks = 0;
  for (int j = 0; j < b.njobs; ++j) {
    b.blk0[j] = blocks;
    blocks += b.job[j].nchunk * b.job[j].B;
  }
  const int s = b.job[0].s;
  const size_t lds = (size_t)s * b.job[0].r * 4;
  if (s <= 8) DPRC_LAUNCH(hpp_rows_batch_kernel<8>, dim3((unsigned)blocks), dim3(kQrThreads), lds, st, b);
  else if (s <= 16) DPRC_LAUNCH(hpp_rows_batch_kernel<16>, dim3((unsigned)blocks), dim3(kQrThreads), lds, st, b);
  else DPRC_LAUNCH(hpp_rows_batch_kernel<32>, dim3((unsigned)blocks), dim3(kQrThreads), lds, st, b);
  return hipGetLastError();
}

hipError_t launch_hpp_sum_batch(const FinalBatch& bt, hipStream_t st) {
  if (bt.njobs < 1 || bt.njobs > kFinMaxJobs) return hipErrorInvalidValue;
  DPRC_LAUNCH(hpp_sum_batch_kernel, dim3((unsigned)bt.job[0].B), dim3(kQrThreads), 0, st, bt);
  return hipGetLastError();
}

int32_t final_chunks(int64_t n) { return (int32_t)ceil_div(n, kFinRows); }

}  // namespace dprc
