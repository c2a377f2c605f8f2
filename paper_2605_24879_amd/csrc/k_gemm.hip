// Clipped accumulation grad = sum_i c_i A_i^T E_i (Algorithm 1, second backward
// pass of a bias-free linear layer) on bf16 matrix cores, fp32 accumulation.
//
// Workgroup tile 256 (d) x 256 (p), eight waves of 128 x 64 (two per SIMD), each a
// 4 x 2 grid of v_mfma_f32_32x32x16_bf16 (128 fp32 accumulators per lane).  The
// contraction runs over tokens and both operands are token-major, so 32-token
// slabs of A and E (256 columns each, 512-byte rows) are loaded with coalesced
// 16-byte buffer reads, two slabs ahead in registers, double-buffered through LDS
// and read back token-contiguous with the LDS transpose read.  Each step is
// software-pipelined over the two 16-token halves of a slab, and the two waves of
// a SIMD cover each other's waits (one wave of 128 x 128 per SIMD with the same
// pipeline, or with LDS reads, writes and loads placed between the MFMAs by
// scheduling barriers, was 7 to 10 percent slower).
//
// Per-sample factors scale the fp32 accumulator at sample boundaries
// (acc <- acc * c_prev / c_i, and * c_last at the end), so the result is
// sum_i c_i (A_i^T E_i) without rounding c_i * E to bf16; samples with c_i = 0
// are skipped.  Tiles are ordered so that the workgroups of one XCD (workgroup
// ids are dealt round-robin to the 8 XCDs) share the tiles of the larger operand.
// Splits over the (sample, slab) list write fp32 partials summed in split order.
#include <algorithm>
#include "device.hpp"
#include "kernels.hpp"

namespace dprc {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;

constexpr int kGM = 256;            // tile rows (d) and columns (p)
constexpr int kGK = 32;             // tokens per slab (64-token slabs measured 5 to 15 percent slower)

__device__ __forceinline__ f32x16_t mfma32x32x16(const uint4& a, const uint4& b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b),
                                                  c, 0, 0, 0);
}

template <int V>
struct GInt {
  static constexpr int value = V;
};

// GM = 256: the 256 x 256 tile `wg` (before the XCD reordering), eight waves of 128 x 64.
// GM = 128: quarter `sub` of that tile, four waves of 64 x 64; three such workgroups share a
// CU.  A quarter's entries are summed in the same order as the whole tile's.  split: the
// token split.
template <int GM, int LD>
__device__ __forceinline__ void gemm_body(const GemmArgs& a, int wg, int split, int sub = 0) {
  constexpr int NW = GM == 256 ? 8 : 4;
  constexpr int kThreads = 64 * NW;
  constexpr int WN = 64, XB = GM == 256 ? 4 : 2;     // wave tile: 32 XB rows, 64 columns
  constexpr int YB = WN / 32;                        // 32-column MFMA blocks per wave
  constexpr int TPR = GM / 8;                        // threads per token row of a slab
  constexpr int RP = kThreads / TPR;                 // slab rows per load pass
  constexpr int RQ = kGK / RP;                       // load passes per slab
  constexpr int kGLd = GM + 32;                      // LDS row: 576 (320) bytes; the 4 rows x 2 column groups of a 32-lane transpose read hit distinct 32-byte bank groups
  __shared__ __attribute__((aligned(16))) uint16_t la[2][kGK * kGLd];
  __shared__ __attribute__((aligned(16))) uint16_t le[2][kGK * kGLd];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int g = lane >> 4, r4 = (lane & 15) >> 2, c4 = lane & 3;
  const int wm = wv / (GM / WN), wn = wv % (GM / WN);     // wave tile rows 32 XB wm, columns 64 wn

  // tile of this workgroup: consecutive ids of one XCD walk the smaller dimension first
  const int tm_n = (a.d + kGM - 1) / kGM, tn_n = (a.p + kGM - 1) / kGM;
  const int ntiles = tm_n * tn_n;
  // a bijection on [0, ntiles) when ntiles is a multiple of 8; identity otherwise
  const int lin = (ntiles & 7) == 0 ? (wg & 7) * (ntiles >> 3) + (wg >> 3) : wg;
  int tm, tn;
  if (a.d <= a.p) { tm = lin % tm_n; tn = lin / tm_n; } else { tn = lin % tn_n; tm = lin / tn_n; }
  const int d0 = tm * kGM + (GM < kGM ? GM * (sub & 1) : 0), p0 = tn * kGM + (GM < kGM ? GM * (sub >> 1) : 0);
  if (GM < kGM && (d0 >= a.d || p0 >= a.p)) return;   // (the whole workgroup)

  const int sps = a.stages_per_sample;
  const int gs_begin = split * a.stages_per_split;
  const int gs_end = min(a.B * sps, gs_begin + a.stages_per_split);
  const int lr = tid / TPR, lc = (tid % TPR) * 8;          // loads: rows lr + RP q, 8 columns at lc
  const int64_t ja = (int64_t)d0 + lc, je = (int64_t)p0 + lc;

  constexpr int NS = 2;                           // slabs in flight
  uint4 ga[NS][RQ], ge[NS][RQ];
  // kLoadVec: per slab one buffer resource per operand over its (up to) 32 token rows,
  // starting at the tile's first column; rows past T and columns past d / p read
  // as zero through out-of-range offsets, and a slab past the sample's last one has
  // an empty range.  kLoadAny: see device.hpp; columns past d / p only reach entries that
  // are not stored, and rows past T are replaced by zeros on the way to LDS.
  const uint32_t arow = (uint32_t)a.lda * 2u, erow = (uint32_t)a.lde * 2u;
  const uint32_t aoff = d0 + lc < a.d ? (uint32_t)lr * arow + 2u * lc : kOobOffset;
  const uint32_t eoff = p0 + lc < a.p ? (uint32_t)lr * erow + 2u * lc : kOobOffset;
  auto gload = [&](int sl, int i, int st, int st_end) __attribute__((always_inline)) {
    const int tok0 = st * kGK;
    const uint16_t* as = a.A + (int64_t)i * a.a_ss;
    const uint16_t* es = a.E + (int64_t)i * a.e_ss;
    if constexpr (LD == kLoadAny) {                // rows past the slab's last read its first
      const int rows = st < st_end ? min(kGK, a.T - tok0) : 0;
      const uint16_t* ab = as + (int64_t)(rows > 0 ? tok0 : 0) * a.lda + d0;
      const uint16_t* eb = es + (int64_t)(rows > 0 ? tok0 : 0) * a.lde + p0;
      const int aroom = operand_room(a.A, a.B, a.T, a.lda, a.d, ab), eroom = operand_room(a.E, a.B, a.T, a.lde, a.p, eb);
#pragma unroll
      for (int r = 0; r < RQ; ++r) {
        const int row = lr + RP * r < rows ? lr + RP * r : 0;
        ga[sl][r] = load16_any(ab, min(aroom, row * (int)a.lda + lc));
        ge[sl][r] = load16_any(eb, min(eroom, row * (int)a.lde + lc));
      }
    } else if constexpr (LD == kLoadVec) {
      const int rows = st < st_end ? min(kGK, a.T - tok0) : 0;
      const int64_t t0 = rows > 0 ? tok0 : 0;
      const __amdgpu_buffer_rsrc_t ar = buffer_rsrc(as + t0 * a.lda + d0, (uint32_t)rows * arow);
      const __amdgpu_buffer_rsrc_t er = buffer_rsrc(es + t0 * a.lde + p0, (uint32_t)rows * erow);
#pragma unroll
      for (int r = 0; r < RQ; ++r) {
        ga[sl][r] = buffer_load16(ar, aoff + (uint32_t)(RP * r) * arow);
        ge[sl][r] = buffer_load16(er, eoff + (uint32_t)(RP * r) * erow);
      }
    } else {
#pragma unroll
      for (int r = 0; r < RQ; ++r) {
        const int t = tok0 + lr + RP * r;
        const bool ok = st < st_end && t < a.T;
        ga[sl][r] = load8_elem(as + (int64_t)(ok ? t : 0) * a.lda, ja, a.d, ok);
        ge[sl][r] = load8_elem(es + (int64_t)(ok ? t : 0) * a.lde, je, a.p, ok);
      }
    }
  };
  // slab st of sample i into LDS buffer buf
  auto swrite = [&](int sl, int buf, int i, int st, int st_end) __attribute__((always_inline)) {
    const int tok0 = st * kGK;
    const int rows = st < st_end ? min(kGK, a.T - tok0) : 0;
    if (LD == kLoadAny && (rows < kGK || d0 + GM > a.d || p0 + GM > a.p)) {
      const int64_t t0 = rows > 0 ? tok0 : 0;
      const int aroom = operand_room(a.A, a.B, a.T, a.lda, a.d, a.A + (int64_t)i * a.a_ss + t0 * a.lda + d0);
      const int eroom = operand_room(a.E, a.B, a.T, a.lde, a.p, a.E + (int64_t)i * a.e_ss + t0 * a.lde + p0);
#pragma unroll
      for (int r = 0; r < RQ; ++r) {
        const bool ok = lr + RP * r < rows;
        const int row = ok ? lr + RP * r : 0;
        const int aat = row * (int)a.lda + lc, eat = row * (int)a.lde + lc;
        const uint4 va = shr_elems(ga[sl][r], aat - min(aat, aroom)), ve = shr_elems(ge[sl][r], eat - min(eat, eroom));
        *reinterpret_cast<uint4*>(&la[buf][(lr + RP * r) * kGLd + lc]) = ok ? va : uint4{0, 0, 0, 0};
        *reinterpret_cast<uint4*>(&le[buf][(lr + RP * r) * kGLd + lc]) = ok ? ve : uint4{0, 0, 0, 0};
      }
      return;
    }
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
      *reinterpret_cast<uint4*>(&la[buf][(lr + RP * r) * kGLd + lc]) = ga[sl][r];
      *reinterpret_cast<uint4*>(&le[buf][(lr + RP * r) * kGLd + lc]) = ge[sl][r];
    }
  };

  f32x16_t acc[XB][YB];
#pragma unroll
  for (int x = 0; x < XB; ++x)
#pragma unroll
    for (int y = 0; y < YB; ++y)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[x][y][q] = 0.f;

  // the lane's transpose-read offsets: rows 8*(g/2) + r4 (+4), columns 16*(g%2) + 4*c4
  const int tr_row = 8 * (g >> 1) + r4, tr_col = 16 * (g & 1) + 4 * c4;
  // The two 16-token halves of a slab are separate register fragment sets (f0, f1):
  // a step multiplies half 0 while reading half 1 and writing the next slab to the
  // other LDS buffer, then (after the step's one barrier) multiplies half 1 while
  // reading half 0 of the next slab, so a wave always has MFMAs whose operands are
  // already in registers.
  uint4 f0a[XB], f0b[YB], f1a[XB], f1b[YB];
  auto frag = [&](uint4 (&av)[XB], uint4 (&bv)[YB], int buf, int ks) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < XB; ++x) {
      const uint16_t* pa = &la[buf][(16 * ks + tr_row) * kGLd + wm * 32 * XB + 32 * x + tr_col];
      av[x] = make_u4(lds_read_tr16(pa), lds_read_tr16(pa + 4 * kGLd));
    }
#pragma unroll
    for (int y = 0; y < YB; ++y) {
      const uint16_t* pe = &le[buf][(16 * ks + tr_row) * kGLd + wn * WN + 32 * y + tr_col];
      bv[y] = make_u4(lds_read_tr16(pe), lds_read_tr16(pe + 4 * kGLd));
    }
  };
  auto mm = [&](const uint4 (&av)[XB], const uint4 (&bv)[YB]) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < XB; ++x)
#pragma unroll
      for (int y = 0; y < YB; ++y) acc[x][y] = mfma32x32x16(av[x], bv[y], acc[x][y]);
  };

  // samples of this split in order; the accumulator is rescaled between samples
  // (outside the slab loop), samples with c_i = 0 are skipped
  float cur_c = 0.f;
  bool started = false;
  const int i_first = gs_begin / sps, i_last = gs_end > gs_begin ? (gs_end - 1) / sps : i_first - 1;
  for (int i = i_first; i <= i_last; ++i) {
    const float ci = a.c[i];
    if (ci == 0.f) continue;
    const int st_lo = max(0, gs_begin - i * sps), st_hi = min(sps, gs_end - i * sps);
    if (started) {
      const float ratio = cur_c / ci;
#pragma unroll
      for (int x = 0; x < XB; ++x)
#pragma unroll
        for (int y = 0; y < YB; ++y) acc[x][y] *= ratio;
    }
    started = true;
    cur_c = ci;
    __syncthreads();                               // the previous sample's last slab is consumed
    // slab k sits in LDS buffer k % 2 while it is multiplied; register slot k % NS
    // receives slab k + NS at the start of that step, and slot (k + 1) % NS (slab
    // k + 1, issued NS - 1 steps earlier) goes to the other buffer at its end.
    // Slabs past the sample's last load empty ranges (zeros).
#pragma unroll
    for (int q = 0; q < NS; ++q) gload(q, i, st_lo + q, st_hi);
    swrite(0, 0, i, st_lo, st_hi);
    __syncthreads();
    frag(f0a, f0b, 0, 0);
    constexpr int NQ = kGK / 16;                 // 16-token quarters of a slab (even)
    auto step = [&](int st, auto u) __attribute__((always_inline)) {
      constexpr int k = decltype(u)::value;      // step index modulo 2 NS
      // loads of slab k + NS (register slot k % NS, free since slab k went to LDS);
      // then the MFMAs of each 16-token part of slab k while reading the next part;
      // slab k + 1 (slot (k + 1) % NS) goes to the other buffer before the barrier,
      // after which the last part is multiplied while part 0 of slab k + 1 is read
      gload(k % NS, i, st + NS, st_hi);
#pragma unroll
      for (int qq = 0; qq + 1 < NQ; ++qq) {
        if (qq % 2 == 0) {
          frag(f1a, f1b, k % 2, qq + 1);
          mm(f0a, f0b);
        } else {
          frag(f0a, f0b, k % 2, qq + 1);
          mm(f1a, f1b);
        }
      }
      swrite((k + 1) % NS, (k + 1) % 2, i, st + 1, st_hi);
      __syncthreads();
      frag(f0a, f0b, (k + 1) % 2, 0);
      mm(f1a, f1b);
    };
    // whole groups of 2 NS steps in the loop (no early exit reaches its back edge,
    // so the compiler's wait counting stays exact), the remainder after it
    int st = st_lo;
    for (; st + 2 * NS <= st_hi; st += 2 * NS) {
      step(st, GInt<0>{});
      step(st + 1, GInt<1>{});
      step(st + 2, GInt<2>{});
      step(st + 3, GInt<3>{});
    }
    if (st < st_hi) step(st, GInt<0>{});
    if (st + 1 < st_hi) step(st + 1, GInt<1>{});
    if (st + 2 < st_hi) step(st + 2, GInt<2>{});
    __syncthreads();                               // the last reads of both buffers are done
  }

  // epilogue: lane holds rows 8*(q/4) + 4*(lane/32) + q%4 and column lane%32 of each 32 x 32 block
  float* dst;
  int64_t ld;
  const bool direct = a.S == 1;
  if (direct) {
    dst = a.out;
    ld = a.ldo;
  } else {
    dst = a.part + (int64_t)split * a.d * a.p;
    ld = a.p;
  }
#pragma unroll
  for (int x = 0; x < XB; ++x)
#pragma unroll
    for (int y = 0; y < YB; ++y) {
      const int col = p0 + wn * WN + 32 * y + (lane & 31);
      if (col >= a.p) continue;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int row = d0 + wm * 32 * XB + 32 * x + 8 * (q >> 2) + 4 * (lane >> 5) + (q & 3);
        if (row >= a.d) continue;
        const float v = acc[x][y][q] * cur_c;
        float* o = dst + (int64_t)row * ld + col;
        if (direct && a.accumulate) *o += v;
        else *o = v;
      }
    }
}

template <int LD>
__global__ __launch_bounds__(512, 1) void gemm_kernel(GemmArgs a) {
  gemm_body<kGM, LD>(a, blockIdx.x, blockIdx.y);
}

// Quarters of the tiles from `first` on, four workgroups each.  (Workgroups go to the XCDs in
// turn, so the quarters of a tile, which share its slabs, sit on four of them, and the order
// of the tiles among the XCDs is not the whole tiles' one.)
template <int LD>
__global__ __launch_bounds__(256) void gemm_quarters_kernel(GemmArgs a, int first) {
  gemm_body<kGM / 2, LD>(a, first + (int)blockIdx.x / 4, 0, (int)blockIdx.x % 4);
}

// Several layers in one launch, each unsplit (S = 1): job j owns blocks blk0[j] ..
// blk0[j] + ntiles_j - 1, and blk0[j] is a multiple of 8, so that a job's blocks are
// dealt to the XCDs as those of a launch of its own; blocks up to the next multiple of
// 8 are idle.  QUARTERS: four workgroups per block, on four XCDs as above.
template <int LD, bool QUARTERS>
__global__ __launch_bounds__(QUARTERS ? 256 : 512, 1) void gemm_batch_kernel(GemmBatch bt) {
  const int blk = QUARTERS ? (int)blockIdx.x / 4 : (int)blockIdx.x;
  int jb = 0;
#pragma unroll 8
  for (int q = 1; q < kGemmMaxJobs; ++q) jb += (q < bt.njobs && blk >= bt.blk0[q]) ? 1 : 0;
  const GemmArgs& a = bt.job[jb];
  const int wg = blk - bt.blk0[jb];
  if (wg >= (int)(((int64_t)a.d + kGM - 1) / kGM * (((int64_t)a.p + kGM - 1) / kGM))) return;
  if constexpr (QUARTERS) gemm_body<kGM / 2, LD>(a, wg, 0, (int)blockIdx.x % 4);
  else gemm_body<kGM, LD>(a, wg, 0);
}

GemmPlan gemm_plan_v2(int64_t B, int64_t T, int64_t d, int64_t p) {
  GemmPlan g;
  g.sps = (int32_t)ceil_div(T, kGK);
  const int64_t total = B * g.sps;
  const int64_t tiles = ceil_div(d, kGM) * ceil_div(p, kGM);
  int64_t S = 1;
  if (tiles < 256) S = std::min<int64_t>(ceil_div(256, tiles), std::max<int64_t>(1, total / 16));
  g.spl = (int32_t)ceil_div(total, S);
  g.S = (int32_t)ceil_div(total, g.spl);
  g.tiles = (int32_t)tiles;
  return g;
}

static int gemm_load(const GemmArgs& a) {        // offsets within one slab stay below 2^31
  return std::min(load_mode(a.vec_a, a.B, a.T, a.d, a.lda, kGK), load_mode(a.vec_e, a.B, a.T, a.p, a.lde, kGK));
}

#define DPRC_GEMM_LOADS(KERNEL, GRID, BLOCK, ...)                                                          \
  if (load == kLoadVec) DPRC_LAUNCH((KERNEL(kLoadVec)), GRID, BLOCK, 0, st, __VA_ARGS__);                  \
  else if (load == kLoadAny) DPRC_LAUNCH((KERNEL(kLoadAny)), GRID, BLOCK, 0, st, __VA_ARGS__);             \
  else DPRC_LAUNCH((KERNEL(kLoadElem)), GRID, BLOCK, 0, st, __VA_ARGS__);

hipError_t launch_gemm(const GemmArgs& a, int64_t ntiles, hipStream_t st) {
  const dim3 grid((unsigned)ntiles, (unsigned)a.S);
  const int load = gemm_load(a);
#define DPRC_K(LD) gemm_kernel<LD>
  DPRC_GEMM_LOADS(DPRC_K, grid, dim3(512), a)
#undef DPRC_K
  return hipGetLastError();
}

hipError_t launch_gemm_quarters(const GemmArgs& a, int64_t first, int64_t ntiles, hipStream_t st) {
  if (a.S != 1 || ntiles < 1 || 4 * ntiles >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(4 * ntiles));
  const int load = gemm_load(a);
#define DPRC_K(LD) gemm_quarters_kernel<LD>
  DPRC_GEMM_LOADS(DPRC_K, grid, dim3(256), a, (int)first)
#undef DPRC_K
  return hipGetLastError();
}

hipError_t launch_gemm_batch(GemmBatch bt, hipStream_t st) {
  if (bt.njobs < 1 || bt.njobs > kGemmMaxJobs) return hipErrorInvalidValue;
  int load = kLoadVec;
  int64_t blocks = 0, tiles = 0;
  for (int j = 0; j < bt.njobs; ++j) {
    const GemmArgs& a = bt.job[j];
    if (a.S != 1) return hipErrorInvalidValue;
    load = std::min(load, gemm_load(a));
    bt.blk0[j] = (int32_t)blocks;
    tiles += ceil_div(a.d, kGM) * ceil_div(a.p, kGM);
    blocks += round_up(ceil_div(a.d, kGM) * ceil_div(a.p, kGM), 8);
  }
  if (4 * blocks >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
  if (tiles <= kGemmQuarterTiles) {
    const dim3 grid((unsigned)(4 * blocks));
#define DPRC_K(LD) gemm_batch_kernel<LD, true>
    DPRC_GEMM_LOADS(DPRC_K, grid, dim3(256), bt)
#undef DPRC_K
  } else {
    const dim3 grid((unsigned)blocks);
#define DPRC_K(LD) gemm_batch_kernel<LD, false>
    DPRC_GEMM_LOADS(DPRC_K, grid, dim3(512), bt)
#undef DPRC_K
  }
#undef DPRC_GEMM_LOADS
  return hipGetLastError();
}

}  // namespace dprc
