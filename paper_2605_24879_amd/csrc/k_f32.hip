// fp32 layers on the fp32 matrix cores (v_mfma_f32_16x16x4_f32: fp32 products and sums):
// the projection Y = X R, the token reduction M = X'^T Y (squared or stored), and the
// clipped accumulation sum_i c_i A_i^T E_i.
//
// Lane layouts of the 16x16x4 MFMA (g = lane / 16, l = lane % 16): A holds row l, k = g;
// B holds k = g, column l; D holds rows 4g .. 4g + 3 of column l.  The token reduction and
// the accumulation contract over tokens, and their operands are token-major, so a lane
// reads W consecutive floats of token row g and uses them as the A (or B) operands of W
// different MFMAs: block x of 16 result rows is then rows W r + x, r < 16, and no operand
// is transposed anywhere.  The projection contracts along the rows of X instead: a lane
// reads 4 consecutive columns of its row and spends them on 4 MFMAs whose k index is
// 4 g + x, with the matching rows of R.
//
// fp32 rows are only 4-byte aligned in general; 16-byte global accesses need no more.
// Pieces that cross the end of a row are read element by element.
#include <algorithm>
#include "device.hpp"
#include "kernels.hpp"

namespace dprc {

template <int V>
struct FInt {
  static constexpr int value = V;
};

template <int W>
struct FVec {
  typedef float type __attribute__((ext_vector_type(W), aligned(4)));
};
typedef FVec<4>::type f4u;

__device__ __forceinline__ f32x4_t mfma_f32(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Four floats at p (columns u .. u + 3 of a row of width lim); columns past lim read as zero.
__device__ __forceinline__ f4u load4_f32(const float* p, int64_t u, int64_t lim) {
  f4u v = {0.f, 0.f, 0.f, 0.f};
  if (u + 4 <= lim) return *reinterpret_cast<const f4u*>(p);
#pragma unroll
  for (int e = 0; e < 3; ++e)
    if (u + e < lim) v[e] = p[e];
  return v;
}

// ---- Y = X R ------------------------------------------------------------------------------
// A workgroup of eight waves (fewer: see the launcher) owns 16 token rows of one sample; the waves take the 64-column
// groups of the width in turn and their partial Y are added in wave order.  The +-1 probe
// words of a chunk of the width are generated into LDS first.  Bound by reading X (a row is
// read once) for up to about 50 columns, by the fp32 matrix rate above.  2048 rows of 4096
// columns and 16 probes took 304 us with one thread per (row, column), 10 us here (3.4 TB/s).
constexpr int kPfWords = 8192;                   // probe words in LDS (32 KB)

template <int NB, int NW>
__global__ __launch_bounds__(64 * NW) void project_f32_kernel(ProjectF32Args a) {
  extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
  uint32_t* zw = smem;                           // [nz][wpc + 1], later the partial tiles
  constexpr int RNB = NB < 4 ? NB : 4;           // column blocks summed per pass over the waves
  float* red = reinterpret_cast<float*>(smem);   // [NW][RNB][16][17]
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const int i = blockIdx.y, t0 = 16 * (int)(blockIdx.z * kFlatGridX + blockIdx.x);
  if (t0 >= a.T) return;
  const int wpc = a.words_per_chunk;             // a multiple of 4
  const int t = t0 + l16;
  const float* x = a.X + (int64_t)i * a.x_ss + (int64_t)(t < a.T ? t : t0) * a.ldx;
  const float* rd = a.nd > 0 ? a.Rd + (int64_t)i * a.r_ss : nullptr;
  f32x4_t acc[NB];
  int zrow[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    acc[nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int cz = 16 * nb + l16 - a.nd;
    zrow[nb] = (cz >= 0 && cz < a.nz ? cz : 0) * (wpc + 1);   // columns past the last are not stored
  }
  auto load = [&](f4u (&v)[4], int u0) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = load4_f32(x + u0 + 16 * q + 4 * g, u0 + 16 * q + 4 * g, a.m);
  };
  for (int uc = 0; uc < a.m; uc += 32 * wpc) {
    const int ncol = min(a.m - uc, 32 * wpc), ngrp = (ncol + 63) / 64;
    f4u cur[4], nxt[4];
    if (wv < ngrp) load(cur, uc + 64 * wv);
    if (a.nz > 0) {
      __syncthreads();                           // the previous chunk's words are used up
      const int nblk = wpc >> 2;
      for (int idx = tid; idx < a.nz * nblk; idx += 64 * NW) {
        const int c = idx / nblk, b = idx - c * nblk;
        const uint32_t w0 = (uint32_t)(uc >> 5) + 4u * (uint32_t)b;
        const u32x4 v = a.probe_kind == kProbeRademacher
            ? rademacher_block(a.key0, a.key1, a.layer_id, a.stream_id, w0 >> 2, (uint32_t)c)
            : u32x4{hadamard_word(w0, c), hadamard_word(w0 + 1, c), hadamard_word(w0 + 2, c), hadamard_word(w0 + 3, c)};
        uint32_t* dst = zw + c * (wpc + 1) + 4 * b;
        dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
      }
      __syncthreads();
    }
    for (int gi = wv; gi < ngrp; gi += NW) {
      const int u0 = uc + 64 * gi;
      if (gi + NW < ngrp) load(nxt, u0 + 64 * NW);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int u = u0 + 16 * q + 4 * g;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          f4u b = {0.f, 0.f, 0.f, 0.f};
          if (a.nz > 0) {
            const uint32_t bits = zw[zrow[nb] + 2 * gi + (q >> 1)] >> (16 * (q & 1) + 4 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) b[e] = __uint_as_float(0x3F800000u | ((bits << (31 - e)) & 0x80000000u));
          }
          if (16 * nb < a.nd) {                  // a block with dense columns (uniform)
            const int c = 16 * nb + l16;
            if (c < a.nd) b = load4_f32(rd + (int64_t)c * a.ld_r + u, u, a.m);
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[nb] = mfma_f32(cur[q][e], b[e], acc[nb]);
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) cur[q] = nxt[q];
    }
  }
  float* y = a.Y + ((int64_t)i * a.T + t0) * a.ncols;
  const int rows = min(16, a.T - t0);
  for (int n0 = 0; n0 < NB; n0 += RNB) {
    __syncthreads();
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      if (nb >= n0 && nb < n0 + RNB)
#pragma unroll
        for (int e = 0; e < 4; ++e) red[((wv * RNB + nb - n0) * 16 + 4 * g + e) * 17 + l16] = acc[nb][e];
    __syncthreads();
    for (int idx = tid; idx < RNB * 256; idx += 64 * NW) {
      const int c = 16 * n0 + idx % (16 * RNB), r = idx / (16 * RNB);
      if (c >= a.ncols || r >= rows) continue;
      const int nb = (idx % (16 * RNB)) >> 4;
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) s += red[((w * RNB + nb) * 16 + r) * 17 + (c & 15)];
      y[(int64_t)r * a.ncols + c] = s;
    }
  }
}

template <int NW>
static hipError_t launch_project_f32_w(const ProjectF32Args& a, hipStream_t st) {
  const int need = (a.ncols + 15) / 16;
  const size_t lds = std::max((size_t)(a.nz > 0 ? a.nz * (a.words_per_chunk + 1) * 4 : 0),
                              (size_t)NW * (need > 2 ? 4 : need) * 16 * 17 * 4);
  const dim3 rows = flat_grid(ceil_div(a.T, 16));
  const dim3 grid(rows.x, (unsigned)a.B, rows.y), blk(64 * NW);
  if (need <= 1) DPRC_LAUNCH((project_f32_kernel<1, NW>), grid, blk, lds, st, a);
  else if (need <= 2) DPRC_LAUNCH((project_f32_kernel<2, NW>), grid, blk, lds, st, a);
  else if (need <= 4) DPRC_LAUNCH((project_f32_kernel<4, NW>), grid, blk, lds, st, a);
  else if (need <= 8) DPRC_LAUNCH((project_f32_kernel<8, NW>), grid, blk, lds, st, a);
  else DPRC_LAUNCH((project_f32_kernel<16, NW>), grid, blk, lds, st, a);
  return hipGetLastError();
}

// Samples that share their columns lie one row stride apart, so short ones share workgroups
// of 16 rows: 3608 one-token samples of 1480 and 8 columns, 350 us in two norm calls of 8
// probes, take 102 us.  A width of 64 (128) columns occupies one (two) of the waves; from
// kManyWgs workgroups on the launch fills the GPU without the others (fewer workgroups are
// faster with all eight: 86 us against 48 for three rows of blocks of 355 tokens).
constexpr int64_t kManyWgs = 512;
hipError_t launch_project_f32(ProjectF32Args a, hipStream_t st) {
  if (a.ncols < 1 || a.ncols > 256 || a.nd + a.nz != a.ncols) return hipErrorInvalidValue;
  if (a.T % 16 != 0 && (a.nd == 0 || a.r_ss == 0) && (int64_t)a.B * a.T <= (1 << 30)) {
    a.T *= a.B;
    a.B = 1;
  }
  a.words_per_chunk = (int32_t)std::min<int64_t>(round_up(ceil_div(a.m, 32), 4),
                                                 a.nz > 0 ? std::max(16, (kPfWords / a.nz) & ~15) : 1 << 24);
  const bool many = ceil_div(a.T, 16) * a.B >= kManyWgs;
  if (many && a.m <= 64) return launch_project_f32_w<1>(a, st);
  if (many && a.m <= 128) return launch_project_f32_w<2>(a, st);
  return launch_project_f32_w<8>(a, st);
}

// ---- M = X^T Y ---------------------------------------------------------------------------------
// A workgroup of eight waves (fewer for short samples) owns 64 result rows (columns of X) and up to 64 result columns
// of one sample; the waves take the token quads in turn, read both operands straight from
// global memory in the MFMA layout, and their partial sums are added in wave order.  The
// result is squared and summed (tilesq) or stored.  Latency-bound at ordinary sizes (512
// tokens are 16 quads per wave): 125 us with one thread per result, 7 us here for a
// 1024-wide operand (its 64 workgroups leave most CUs idle) and 9 us for a 4096-wide one.
constexpr int kTfTile = 64;

template <int NB, int NW>
__global__ __launch_bounds__(64 * NW) void tokred_f32_kernel(TokredF32Args a) {
  constexpr int U = 4;                           // token quads in flight per wave
  __shared__ float red[NW][kTfTile][17];
  __shared__ double dred[NW];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const int tn = (a.ncols + 16 * NB - 1) / (16 * NB);              // tiles of columns
  const int jt = (int)(blockIdx.y / tn * kFlatGridX + blockIdx.x), ct = blockIdx.y % tn, i = blockIdx.z;
  const int j0 = kTfTile * jt, c0 = 16 * NB * ct;
  if (j0 >= a.n) return;
  const float* xs = a.X + (int64_t)i * a.x_ss + j0 + 4 * l16;
  const float* ys = a.Y + (int64_t)i * a.T * a.ncols;
  int ycol[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) ycol[nb] = min(c0 + 16 * nb + l16, a.ncols - 1);
  f32x4_t acc[4][NB];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[x][nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int nq = (a.T + 3) / 4;
  for (int q0 = wv; q0 < nq; q0 += U * NW) {
    f4u xv[U];
    float yv[U][NB];
#pragma unroll
    for (int u = 0; u < U; ++u) {                // tokens past the last add zeros
      const int t = 4 * (q0 + u * NW) + g;
      const int64_t tt = t < a.T ? t : 0;
      xv[u] = load4_f32(xs + tt * a.ldx, j0 + 4 * l16, t < a.T ? a.n : 0);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const float y = ys[tt * a.ncols + ycol[nb]];
        yv[u][nb] = t < a.T ? y : 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[x][nb] = mfma_f32(xv[u][x], yv[u][nb], acc[x][nb]);
  }
  double sq = 0.0;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[wv][4 * (4 * g + e) + x][l16] = acc[x][nb][e];
    __syncthreads();
    for (int idx = tid; idx < kTfTile * min(16, a.ncols - c0 - 16 * nb); idx += 64 * NW) {
      const int jl = idx % kTfTile, cl = idx / kTfTile, c = c0 + 16 * nb + cl, j = j0 + jl;
      if (j >= a.n) continue;
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) s += red[w][jl][cl];
      if (a.M) a.M[(int64_t)i * a.m_ss + (int64_t)c * a.m_ld + j] = s;
      else sq += (double)s * (double)s;
    }
  }
  if (a.M) return;
  sq = wave_sum(sq);
  if (lane == 0) dred[wv] = sq;
  __syncthreads();
  if (tid == 0) {
    double s = 0.0;
    for (int w = 0; w < NW; ++w) s += dred[w];
    a.tilesq[((int64_t)i * tn + ct) * ((a.n + kTfTile - 1) / kTfTile) + jt] = s;
  }
}

// Columns per workgroup: 64 share one read of X, fewer when there are fewer.
static int tokred_f32_nb(int32_t ncols) { return ncols <= 16 ? 1 : (ncols <= 32 ? 2 : 4); }

int32_t tokred_f32_tiles(int64_t n, int32_t ncols) {
  return (int32_t)(ceil_div(n, kTfTile) * ceil_div(ncols, 16 * tokred_f32_nb(ncols)));
}

template <int NW>
static hipError_t launch_tokred_f32_w(const TokredF32Args& a, hipStream_t st) {
  const int nb = tokred_f32_nb(a.ncols);
  const dim3 rows = flat_grid(ceil_div(a.n, kTfTile));
  const dim3 grid(rows.x, rows.y * (unsigned)ceil_div(a.ncols, 16 * nb), (unsigned)a.B);
  const dim3 blk(64 * NW);
  if (nb == 1) DPRC_LAUNCH((tokred_f32_kernel<1, NW>), grid, blk, 0, st, a);
  else if (nb == 2) DPRC_LAUNCH((tokred_f32_kernel<2, NW>), grid, blk, 0, st, a);
  else DPRC_LAUNCH((tokred_f32_kernel<4, NW>), grid, blk, 0, st, a);
  return hipGetLastError();
}

// Short samples leave most of eight waves without token quads, and what is left of their work
// is the sum over the waves: up to 16 tokens (one step of one wave) a workgroup is one wave,
// up to 256 two, if there are enough workgroups to fill the GPU without the others.  1979
// samples of 11 tokens, 4248 > 8, one probe: 507 us with eight waves, 108 with one; 307 of
// 34 tokens, 2344 > 584, 32 probes: 222 and 121 with two.  At 385 tokens two were 17% slower.
hipError_t launch_tokred_f32(const TokredF32Args& a, hipStream_t st) {
  if (a.ncols < 1 || (!a.M && !a.tilesq)) return hipErrorInvalidValue;
  const bool many = (int64_t)a.B * tokred_f32_tiles(a.n, a.ncols) >= kManyWgs;
  if (many && a.T <= 16) return launch_tokred_f32_w<1>(a, st);
  if (many && a.T <= 256) return launch_tokred_f32_w<2>(a, st);
  return launch_tokred_f32_w<8>(a, st);
}

// ---- sum_i c_i A_i^T E_i ----------------------------------------------------------------------
// MW x NW x KS waves: MW x NW of them share a tile of 16 W MW x 16 W NW, KS of them each
// take 1/KS of the token quads of a slab and their sums are added in order at the end
// (128-wide tiles: two waves per SIMD; smaller tiles, for outputs too small to give every CU
// a large one: four waves on one accumulator tile).  32-token slabs of A and E go through
// double-buffered LDS, two slabs ahead in registers.  Each sample is summed by itself and
// then added, scaled by its factor; samples with factor 0 are skipped.  Bound by the fp32
// matrix rate (157 TFLOP/s) from 256 tiles up: 1024 x 4096 over 2048 tokens took 4144 us with
// one thread per entry and takes 168 us here (102 TFLOP/s).  When it took 177, slabs of 16
// tokens measured 194 us, 128 x 64 tiles of four waves with two workgroups per CU 189, the
// 32x32x2 MFMA 196, fragment reads pinned ahead of the MFMAs 176.  One to four tokens in all
// over more than 256 tiles are bound by the stores of the second round (1027 x 4097: 17 us, 10
// with one thread per entry; 27 with 64-wide tiles).
constexpr int kFK = 32;                          // tokens per slab

// NARROW: operands less than 4 wide (or strides past 32-bit offsets), read by element.
// PACKED, for samples of at most 16 tokens (half a slab): a slab holds several samples, each on
// as many of its token quads (1, 2 or 4) as it needs.  A sample's sum is still formed by
// itself and scaled as a whole; rows of samples with factor 0 become zeros.  128 one-token
// samples of 1024 > 1024: 64 us with one thread per entry, 207 with a slab per sample, 40 here;
// of 16 tokens 1017, 198 and 142.
template <int W, int MW, int NW, int KS, bool NARROW, bool PACKED>
__global__ __launch_bounds__(64 * MW * NW * KS) void gemm_f32_kernel(GemmF32Args a) {
  constexpr int TM = 16 * W * MW, TN = 16 * W * NW;
  constexpr int NT = 64 * MW * NW * KS;
  constexpr int NA = kFK * TM / 4 / NT, NP = NA + kFK * TN / 4 / NT;   // 16-byte pieces per thread and slab: A, A and E
  constexpr int KQ = kFK / 4 / KS;               // token quads per wave and slab
  typedef float vec __attribute__((ext_vector_type(W)));
  __shared__ __attribute__((aligned(16))) float la[2][kFK][TM];
  __shared__ __attribute__((aligned(16))) float le[2][kFK][TN];
  __shared__ float red[MW * NW * KS][16][16 * W + 1];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const int kg = wv / (MW * NW), wi = wv % (MW * NW), kgu = __builtin_amdgcn_readfirstlane(kg);
  const int tn_n = (a.p + TN - 1) / TN;
  const int d0 = (int)(blockIdx.x / tn_n) * TM, p0 = (int)(blockIdx.x % tn_n) * TN;
  const int wm = (wi / NW) * 16 * W, wn = (wi % NW) * 16 * W;
  // PACKED: 1 << lq quads per sample, kFK / 4 >> lq samples per slab
  const int lq = a.T <= 4 ? 0 : (a.T <= 8 ? 1 : 2), per_slab = (kFK / 4) >> lq;
  const int sps = PACKED ? (a.B + per_slab - 1) / per_slab : (a.T + kFK - 1) / kFK;
  // piece r of this thread: operand A for r < NA, else E; token row and column of the
  // slab.  A piece that would cross the end of its row starts at width - 4 instead and is
  // shifted down in registers; one past the end is the row's last, and what it brings only
  // reaches entries that are not stored.
  int prow[NP], lrow[NP], pcol[NP], psh[NP], psam[PACKED ? NP : 1];   // prow in memory, lrow in LDS
  int32_t poff[NP];
  constexpr int kNoRow = 1 << 30;                // an LDS row that no token has
#pragma unroll
  for (int r = 0; r < NP; ++r) {
    const int id = tid + NT * (r < NA ? r : r - NA), ppr = (r < NA ? TM : TN) / 4;
    prow[r] = lrow[r] = id / ppr;
    pcol[r] = 4 * (id % ppr);
    if constexpr (PACKED) {
      psam[r] = lrow[r] >> (2 + lq);
      const int t = lrow[r] & ((4 << lq) - 1);
      prow[r] = t < a.T ? psam[r] * a.T + t : kNoRow;
    }
    const int room = (r < NA ? a.d - d0 : a.p - p0) - 4;     // the last start of a whole piece
    psh[r] = NARROW ? 0 : min(3, max(0, pcol[r] - room));
    poff[r] = NARROW ? 0 : 4 * ((int32_t)((prow[r] < kNoRow ? prow[r] : 0) * (r < NA ? a.lda : a.lde)) + min(pcol[r], room));
  }
  f4u ring[2][NP];
  float fac[2][PACKED ? NP : 1];                 // the factors of the pieces' samples
  int rows[2];                                   // token rows of the slabs in the ring
  // Every step issues the same loads (past the last slab: that slab again), so that the
  // waits on the in-order load counter count exactly.
  auto gload = [&](f4u (&dst)[NP], float (&f)[PACKED ? NP : 1], int& nrow, int i, int st) __attribute__((always_inline)) {
    const int64_t row0 = PACKED ? (int64_t)st * per_slab * a.T : (int64_t)st * kFK;
    const float* ab = a.A + (int64_t)i * a.a_ss + row0 * a.lda + d0;
    const float* eb = a.E + (int64_t)i * a.e_ss + row0 * a.lde + p0;
    nrow = PACKED ? min(per_slab, a.B - st * per_slab) * a.T : min(kFK, a.T - st * kFK);
#pragma unroll
    for (int r = 0; r < NP; ++r) {
      const bool ok = prow[r] < nrow;
      if constexpr (PACKED) f[r] = a.c[min(st * per_slab + psam[r], a.B - 1)];
      if constexpr (NARROW) {
        dst[r] = load4_f32((r < NA ? ab : eb) + (int64_t)(ok ? prow[r] : 0) * (r < NA ? a.lda : a.lde) + pcol[r],
                           (r < NA ? d0 : p0) + pcol[r], ok ? (r < NA ? a.d : a.p) : 0);
      } else {                                   // a row past the sample reads the slab's first
        const int32_t back = 4 * (int32_t)((prow[r] < kNoRow ? prow[r] : 0) * (r < NA ? a.lda : a.lde));
        dst[r] = *reinterpret_cast<const f4u*>(reinterpret_cast<const char*>(r < NA ? ab : eb) +
                                               (ok ? poff[r] : poff[r] - back));
      }
    }
  };
  auto swrite = [&](const f4u (&src)[NP], const float (&f)[PACKED ? NP : 1], int nrow, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < NP; ++r) {
      f4u v = src[r];
      if (!NARROW) {
        if (psh[r] & 1) v = f4u{v[1], v[2], v[3], v[3]};
        if (psh[r] & 2) v = f4u{v[2], v[3], v[3], v[3]};
      }
      const bool ok = prow[r] < nrow && !(PACKED && f[PACKED ? r : 0] == 0.f);   // rows past the sample add zeros
      *reinterpret_cast<float4*>(r < NA ? &la[buf][lrow[r]][pcol[r]] : &le[buf][lrow[r]][pcol[r]]) =
          float4{ok ? v[0] : 0.f, ok ? v[1] : 0.f, ok ? v[2] : 0.f, ok ? v[3] : 0.f};
    }
  };
  f32x4_t acc[W][W], tot[W][W];
#pragma unroll
  for (int x = 0; x < W; ++x)
#pragma unroll
    for (int y = 0; y < W; ++y) acc[x][y] = tot[x][y] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto next_sample = [&](int i) {                // first sample >= i with a factor other than zero
    if (PACKED) return i > 0 ? a.B : 0;          // (all of them in one)
    while (i < a.B && a.c[i] == 0.f) ++i;
    return i;
  };
  // (li, ls): the slab to load next, at most the last one; (ci, cs): the slab to multiply
  int li = next_sample(0), ls = 0, ci = li, cs = 0;
  auto advance = [&](int& i, int& st) __attribute__((always_inline)) {
    if (++st == sps) {
      st = 0;
      i = next_sample(i + 1);
    }
  };
  auto load_next = [&](int slot) __attribute__((always_inline)) {
    gload(ring[slot], fac[slot], rows[slot], li, ls);
    int i = li, st = ls;
    advance(i, st);
    if (i < a.B) {
      li = i;
      ls = st;
    }
  };
  vec fa[2], fe[2];
  auto frag = [&](vec& av, vec& ev, int buf, int ks) __attribute__((always_inline)) {
    const int k = 4 * (KQ * kg + ks) + g;
    av = *reinterpret_cast<const vec*>(&la[buf][k][wm + W * l16]);
    ev = *reinterpret_cast<const vec*>(&le[buf][k][wn + W * l16]);
  };
  auto mm = [&](const vec& av, const vec& ev) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < W; ++x)
#pragma unroll
      for (int y = 0; y < W; ++y) acc[x][y] = mfma_f32(av[x], ev[y], acc[x][y]);
  };
  auto fold = [&](float f) __attribute__((always_inline)) {          // a sample's sum joins the total
#pragma unroll
    for (int x = 0; x < W; ++x)
#pragma unroll
      for (int y = 0; y < W; ++y)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          tot[x][y][e] = fmaf(f, acc[x][y][e], tot[x][y][e]);
          acc[x][y][e] = 0.f;
        }
  };
  // PACKED: after quad ks of this wave, the last of its sample here
  auto fold_quad = [&](int ks) __attribute__((always_inline)) {
    const int fq = min(1 << lq, KQ);
    if (PACKED && ((ks + 1) & (fq - 1)) == 0) fold(a.c[min(cs * per_slab + ((KQ * kgu + ks) >> lq), a.B - 1)]);
  };
  auto step = [&](auto b) __attribute__((always_inline)) {
    constexpr int buf = decltype(b)::value;
    // ring slot `buf` held the slab now in LDS buffer `buf`; the other slot holds the next
    load_next(buf);
    // the fragments of a quad are read while the one before is multiplied, those of the next
    // slab's first quad (after the step's one barrier) while the last is
#pragma unroll
    for (int ks = 0; ks + 1 < KQ; ++ks) {
      frag(fa[(ks + 1) & 1], fe[(ks + 1) & 1], buf, ks + 1);
      mm(fa[ks & 1], fe[ks & 1]);
      fold_quad(ks);
    }
    swrite(ring[buf ^ 1], fac[buf ^ 1], rows[buf ^ 1], buf ^ 1);
    __syncthreads();
    if constexpr (KQ % 2 == 0) {
      frag(fa[0], fe[0], buf ^ 1, 0);
      mm(fa[1], fe[1]);
    } else {
      mm(fa[0], fe[0]);
      frag(fa[0], fe[0], buf ^ 1, 0);
    }
    if constexpr (PACKED) fold_quad(KQ - 1);
    else if (cs + 1 == sps) fold(a.c[ci]);       // the sample's last slab
    advance(ci, cs);
  };
  if (ci < a.B) {
    load_next(0);
    load_next(1);
    swrite(ring[0], fac[0], rows[0], 0);
    __syncthreads();
    frag(fa[0], fe[0], 0, 0);
    while (ci < a.B) {
      step(FInt<0>{});
      if (ci >= a.B) break;
      step(FInt<1>{});
    }
  }
  // a lane's entries: rows wm + W (4 g + e) + x, columns wn + W l16 + y of the tile.  Block x
  // of every wave goes through LDS, and the KS sums of an entry are added in order.
  constexpr int NC = 16 * W / (4 * KS), V = NC < 4 ? NC : 4;   // columns per thread and block x, per store
  const int tw = tid / (64 * KS), tr = tid % (64 * KS) / (4 * KS), tc = V * (tid % (4 * KS));
  for (int x = 0; x < W; ++x) {
    __syncthreads();
#pragma unroll
    for (int xx = 0; xx < W; ++xx)
      if (xx == x)
#pragma unroll
        for (int y = 0; y < W; ++y)
#pragma unroll
          for (int e = 0; e < 4; ++e) red[wv][4 * g + e][W * l16 + y] = tot[xx][y][e];
    __syncthreads();
    const int row = d0 + (tw / NW) * 16 * W + W * tr + x;
    if (row >= a.d) continue;
#pragma unroll
    for (int c = tc; c < 16 * W; c += V * 4 * KS) {            // the threads of a row store next to each other
      const int col = p0 + (tw % NW) * 16 * W + c;
      float* o = a.out + (int64_t)row * a.ldo + col;
      typename FVec<V>::type v;
#pragma unroll
      for (int n = 0; n < V; ++n) {
        v[n] = red[tw][tr][c + n];
#pragma unroll
        for (int q = 1; q < KS; ++q) v[n] += red[q * MW * NW + tw][tr][c + n];
      }
      if (col + V <= a.p) {
        auto* ov = reinterpret_cast<typename FVec<V>::type*>(o);
        *ov = a.accumulate ? *ov + v : v;
      } else {
#pragma unroll
        for (int n = 0; n < V; ++n)
          if (col + n < a.p) o[n] = a.accumulate ? o[n] + v[n] : v[n];
      }
    }
  }
}

// The largest tile that still gives every CU a workgroup.
template <bool NARROW, bool PACKED>
static hipError_t launch_gemm_f32_n(const GemmF32Args& a, hipStream_t st) {
  auto tiles = [&](int64_t m, int64_t n) { return ceil_div(a.d, m) * ceil_div(a.p, n); };
  if (tiles(128, 128) >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
  if (tiles(128, 128) >= 256)
    DPRC_LAUNCH((gemm_f32_kernel<4, 2, 2, 2, NARROW, PACKED>), dim3((unsigned)tiles(128, 128)), dim3(512), 0, st, a);
  else if (tiles(64, 64) >= 256)
    DPRC_LAUNCH((gemm_f32_kernel<4, 1, 1, 4, NARROW, PACKED>), dim3((unsigned)tiles(64, 64)), dim3(256), 0, st, a);
  else
    DPRC_LAUNCH((gemm_f32_kernel<2, 1, 1, 4, NARROW, PACKED>), dim3((unsigned)tiles(32, 32)), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_gemm_f32(const GemmF32Args& a, hipStream_t st) {
  const bool narrow = a.d < 4 || a.p < 4 || std::max(a.lda, a.lde) >= ((int64_t)1 << 23);
  const bool packed = a.B > 1 && a.T <= 16;
  if (packed) return narrow ? launch_gemm_f32_n<true, true>(a, st) : launch_gemm_f32_n<false, true>(a, st);
  return narrow ? launch_gemm_f32_n<true, false>(a, st) : launch_gemm_f32_n<false, false>(a, st);
}

}  // namespace dprc
