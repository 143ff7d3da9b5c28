// Fused, never-materialised kernel-matrix products for gfx950.
//
//   square:  W = K_hat V = s_f M(X, X) V + sigma^2 V,  M_ab = m(r_ab)
//   cross:   W = K(Z, X) V = s_f M(Z, X) V
//
// with r_ab^2 = sum_j ((x_aj - x_bj)/l_j)^2 and m the Matern-5/2 or RBF
// profile (the kernel of Sec. 4; K_hat of Sec. 2.2; the O(N^2) product that
// CG needs, Sec. 3.1, never stored, Sec. 3.2).
//
// One workgroup = 4 wave64s, each owning 16*NA output rows a.  A wave keeps
// the MFMA fragments of its rows in registers and sweeps the b stream in
// chunks of 32 points.  Per (16-row block, 32-point chunk):
//   1. S = XR_b . XC_a^T on the matrix cores gives r^2 directly: the operands
//      carry -2 x~_b against x~_a plus the two squared norms folded into the
//      K padding, so no VALU work builds the distance.
//   2. m(r) is evaluated in registers on the S accumulator (v_sqrt, v_exp,
//      two FMAs); the accumulator layout (lane = a, 4 consecutive b per lane
//      group) is already the A-operand layout of the next product once the
//      K index of that product is permuted to match, so nothing goes through
//      LDS.
//   3. acc += M . V_b on the matrix cores.
// FP32 accumulators are flushed to FP64 every FLUSH chunks.  The diagonal
// element of the square product is masked out of the tiles and added exactly
// in FP64 by the epilogue as (s_f + sigma^2) V.
//
// Two arithmetic forms share this structure:
//   BF16X3 (the mixed form; the name is the ABI's): the distance from FP16
//           hi/lo coordinates (centred on the b stream's column means) with the
//           three products hi.hi + hi.lo + lo.hi on v_mfma_f32_16x16x32_f16; M
//           and V split x = hi + lo in FP16 as well, after power-of-two scalings
//           that keep them in FP16's normal range (2^15 M; each column of V so
//           that its largest entry lies in [2^14, 2^15)), the same three
//           products on the same instruction; FP32 accumulation, the scalings
//           undone exactly in the FP64 epilogue.
//   FP32:   v_mfma_f32_16x16x4_f32 for both products; the squared norms
//           initialise the distance accumulator.
// Row-independent BF16X3 cross products with many columns (prediction) use a
// variant that evaluates each entry once for all columns (the wide sweep),
// described where it is defined; the FP64 form (low-noise regime) is in
// kmm_fp64.hip.
#include "internal.h"
#include "mfma_bf16.h"
#include "reduce.h"

#include <algorithm>
#include <mutex>
#include <vector>
#include <cmath>

namespace gpk {

constexpr int kFlush = 32;  // 32-point chunks accumulated in FP32 before the FP64 flush
constexpr int kF64MaxD = 64;   // FP64 form: features held in registers

// The profile m(r) from S = r^2 scaled as above.  ACCURATE replaces the raw
// v_sqrt_f32 by v_rsq_f32 plus one Newton step on the residual S - u^2.  The raw
// instruction is within 9.3e-8 relative (about 1.6 ulp; 15% of results not
// correctly rounded, slightly biased low) and the Newton form correctly rounded,
// both measured over 4.2M values in [1e-2, 1e3).  The FP32 form uses the Newton
// form (its VALU work hides behind the slower FP32 matrix cores); in the mixed
// form the hi/lo splits dominate the error.
template <int KIND, bool ACCURATE>
__device__ __forceinline__ float profile(float S) {
  if constexpr (KIND == GP_MATERN52) {
    float u;
    if constexpr (ACCURATE) {
      const float s = __builtin_fmaxf(__builtin_fabsf(S), 1e-30f);
      const float y = __builtin_amdgcn_rsqf(s);
      const float u0 = s * y;
      u = __builtin_fmaf(__builtin_fmaf(-u0, u0, s), 0.5f * y, u0);
    } else {
      u = __builtin_amdgcn_sqrtf(__builtin_fabsf(S));
    }
    const float e = __builtin_amdgcn_exp2f(-u);
    const float poly = __builtin_fmaf(__builtin_fmaf(u, kMaternC2, kMaternC1), u, 1.0f);
    return poly * e;
  } else {
    return __builtin_amdgcn_exp2f(-__builtin_fabsf(S));
  }
}

// kMScale m(r) for the mixed form's FP16 value products: the Matern scale rides in
// the polynomial's constants, the RBF one costs a multiply.
template <int KIND>
__device__ __forceinline__ float profile_scaled(float S) {
  if constexpr (KIND == GP_MATERN52) {
    const float u = __builtin_amdgcn_sqrtf(__builtin_fabsf(S));
    const float e = __builtin_amdgcn_exp2f(-u);
    return __builtin_fmaf(__builtin_fmaf(u, kMaternC2s, kMaternC1s), u, kMScale) * e;
  } else {
    return __builtin_amdgcn_exp2f(-__builtin_fabsf(S)) * kMScale;
  }
}

// ---------------------------------------------------------------- preparation
//
// Distances of the mixed form.  r^2 = n_a + n_b - 2 x'_a . x'_b runs on the FP16
// matrix cores with each centred, scaled coordinate x' = (x - c) s split as
// x' ~ h + l, h = RNE16(x'), l = RNE16(x' - h) (22 significant bits), and the
// three products h.h + h.l + l.h; n = sum (h + l)^2, so that the dropped l.l
// leaves an error of 2 l_a . l_b (about 2^-22 |x'|^2, of either sign) instead of a
// bias.  The centre c is the column mean of the b stream (the training points),
// so the coordinates, and with them the cancellation in n_a + n_b - 2 x'_a . x'_b,
// stay as small as the data's spread allows whatever its offset.  FP16 holds
// |h| <= 32752 (-2h must stay finite): a point with a scaled coordinate beyond
// that, about 10^4 lengthscales from the centre, gets a NaN norm, and every
// product involving it is NaN (never silently wrong).  The norms enter the K
// padding as three FP16 digits against the constants kNormScale (a mixed-radix
// expansion whose residual is below 1e-9 relative up to n ~ 2e9).

constexpr float kNormScale[3] = {32768.f, 16.f, 0.0078125f};  // 2^15, 2^4, 2^-7
constexpr double kMaxScaled = 32752.0;                      // largest |h| with -2h finite in FP16
constexpr double kMaxNorm = 65504.0 * 32768.0;              // largest n the top digit holds

__device__ __forceinline__ double f16_round(double x) { return (double)(_Float16)(float)x; }

// Column means of the row-major n x d matrix X (the centre of the mixed form), in
// two fixed-order passes: sums over blocks of consecutive rows, then over the
// blocks, so that repeated runs give the same bits.
constexpr int64_t kMeanBlocks = 1024;

static int64_t colmean_blocks(int64_t n) {
  return std::max<int64_t>(1, std::min<int64_t>(kMeanBlocks, (n + 255) / 256));
}

size_t colmean_scratch_doubles(int64_t n, int d) { return (size_t)colmean_blocks(n) * (size_t)d; }

// Both passes add in order; their loads are issued 32 rows (or all blocks) ahead,
// since one load at a time made the second pass 244 us at n = 262,144 (10 us now).
__device__ __forceinline__ void colmean_partial(const double* __restrict__ X, int64_t n, int d, int64_t rows_per_blk,
                                                int64_t blk, double* __restrict__ part) {
  const int j = threadIdx.x;
  if (j >= d) return;
  const int64_t r0 = blk * rows_per_blk;
  const int64_t r1 = r0 + rows_per_blk < n ? r0 + rows_per_blk : n;
  double s = 0.0;
  int64_t i = r0;
  for (; i + 32 <= r1; i += 32) {
    double v[32];
#pragma unroll
    for (int u = 0; u < 32; ++u) v[u] = X[(i + u) * d + j];
#pragma unroll
    for (int u = 0; u < 32; ++u) s += v[u];
  }
  for (; i < r1; ++i) s += X[i * d + j];
  part[blk * d + j] = s;
}

__global__ __launch_bounds__(128) void colmean_partial_kernel(const double* __restrict__ X, int64_t n, int d,
                                                              int64_t rows_per_blk, double* __restrict__ part) {
  colmean_partial(X, n, d, rows_per_blk, blockIdx.x, part);
}

constexpr int kMeanCols = 8;  // columns per workgroup of the second pass

__global__ __launch_bounds__(256) void colmean_final_kernel(const double* __restrict__ part, int nblk, int d, int64_t n,
                                                            double* __restrict__ mu) {
  __shared__ double p[kMeanCols][kMeanBlocks + 1];
  const int j0 = blockIdx.x * kMeanCols;
  constexpr int kPer = kMeanCols * (int)kMeanBlocks / 256;
  const int jl = threadIdx.x % kMeanCols, bl = threadIdx.x / kMeanCols;
  const int j = j0 + jl < d ? j0 + jl : d - 1;
  double v[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int b = bl + 256 / kMeanCols * u;
    if (256 / kMeanCols * u < nblk) v[u] = part[(int64_t)(b < nblk ? b : nblk - 1) * d + j];
  }
#pragma unroll
  for (int u = 0; u < kPer; ++u) p[jl][bl + 256 / kMeanCols * u] = v[u];
  __syncthreads();
  if (threadIdx.x >= kMeanCols || j0 + (int)threadIdx.x >= d) return;
  const double* const q = p[threadIdx.x];
  double s = 0.0;
  int b = 0;
  for (; b + 16 <= nblk; b += 16) {
    double w[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) w[u] = q[b + u];
#pragma unroll
    for (int u = 0; u < 16; ++u) s += w[u];
  }
  for (; b < nblk; ++b) s += q[b];
  mu[j0 + threadIdx.x] = s / (double)n;
}

hipError_t column_means(const double* X, int64_t n, int d, double* part, double* mu, hipStream_t st) {
  if (!X || !part || !mu || n < 1 || d < 1 || d > GP_MAX_D) return hipErrorInvalidValue;
  const int64_t nblk = colmean_blocks(n);
  const int64_t rpb = (n + nblk - 1) / nblk;
  colmean_partial_kernel<<<(unsigned)nblk, 128, 0, st>>>(X, n, d, rpb, part);
  colmean_final_kernel<<<(unsigned)((d + kMeanCols - 1) / kMeanCols), 256, 0, st>>>(part, (int)nblk, d, n, mu);
  return hipGetLastError();
}

// Squared norm of each prepared point of the FP32 form: n = sum f^2 in FP64 with
// f = fl32(x s), no centring.
__global__ __launch_bounds__(256) void prep_norm_fp32_kernel(const double* __restrict__ X, int64_t n, int64_t npad,
                                                             int d, Scale sc, double* __restrict__ nrm) {
  // Each wave owns 64 consecutive points.  Per slice of 16 features the wave
  // loads the 64 x 16 block of X (each load instruction covers four rows'
  // 128-byte runs), turns every element into its norm term and parks the terms
  // in LDS; lane r then adds row r's terms in feature order, the same sequence
  // of additions as a per-point loop over the features.
  constexpr int kF = 16;
  __shared__ double term[4][64][kF + 1];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t r0 = ((int64_t)blockIdx.x * 4 + wave) * 64;
  const int fl = lane & 15;
  double s = 0.0;
  if (n > 0) {  // the same for the whole block
    for (int j0 = 0; j0 < d; j0 += kF) {
      const int f = j0 + fl < d ? j0 + fl : d - 1;
      const double scale = sc.s[f];
      double x[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) {  // row 4 k + lane / 16 of the wave's 64 (clamped into X)
        const int64_t pr = r0 + 4 * k + (lane >> 4);
        x[k] = X[(pr < n ? pr : n - 1) * d + f];
      }
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const int i = 4 * k + (lane >> 4);
        const double fv = (float)(x[k] * scale);
        term[wave][i][fl] = (r0 + i < n && j0 + fl < d) ? fv * fv : 0.0;
      }
      __syncthreads();
      const int nf = d - j0 < kF ? d - j0 : kF;
      for (int q = 0; q < nf; ++q) s += term[wave][lane][q];
      __syncthreads();  // the next slice overwrites the terms
    }
  }
  const int64_t p = r0 + lane;
  if (p < npad) nrm[p] = p < n ? s : 0.0;
}

// Mixed-form point fragments.  K layout of a prepared point (length 32*KS, zero padded):
//   row side (b):    [-2h_0..-2h_{d-1}, -2h_0.., -2l_0.., D2, D1, D0, C2, C1, C0, 0..]
//   column side (a): [  h_0..  h_{d-1},   l_0..,   h_0.., C2, C1, C0, D2, D1, D0, 0..]
// with C = kNormScale and D the point's norm digits (n = sum_k D_k C_k), so that
// sum_K row*col = -2(h.h + h.l + l.h) + n_b + n_a.  FP16 values, stored as
// 16-byte units.  Fragment (blk, ks, lane) holds K = 32 ks + 8 (lane/16) + j,
// j = 0..7, of point 16 blk + lane%16.  nrm (nullable): the squared norms.
//
// Bound by HBM: X read once, both sides written once.  A workgroup builds the K
// rows of 32 points in LDS: every thread splits two elements of each 16-feature
// slice of X (128-byte runs, all slices loaded ahead) and scatters the halves, one
// thread per point adds the norm in feature order and appends the digits, and the rows leave as 16-byte units in fragment
// order.  n = 262,144, d = 48: 34 us for the norms plus 215 us for the fragments,
// whose threads each found their eight K values by division and split them anew;
// 55 us here.
constexpr int kPrepPts = 32;

// The centre: given, or (part) the column sums of nblk <= kMeanFold blocks, added and
// divided as in colmean_final_kernel and stored to ctr by the first workgroup.
constexpr int kMeanFold = 16;

struct PointSet {
  const double* X;
  int64_t n;          // points; rows beyond them are padding
  bf16x8 *xr, *xc;    // row and column side (nullable)
  double* nrm;        // nullable
};

struct Centre {
  double* ctr;
  const double* part;  // null: ctr holds the centre
  int nblk;
  int64_t n;
};

template <int NS>  // 16-feature slices
__device__ __forceinline__ void prep_points_block(const PointSet& ps, const Centre& ce, int64_t blk, int d, int KS,
                                                  const Scale& sc) {
  extern __shared__ __attribute__((aligned(16))) _Float16 rows[];  // [side][point][pitch]
  __shared__ int bad[kPrepPts];
  __shared__ double cm[GP_MAX_D];
  const double* __restrict__ X = ps.X;
  const int64_t n = ps.n;
  bf16x8* __restrict__ xr = ps.xr;
  bf16x8* __restrict__ xc = ps.xc;
  double* __restrict__ nrm = ps.nrm;
  const int pitch = 32 * KS + 8;  // halves
  _Float16* const Rr = rows;
  _Float16* const Rc = rows + kPrepPts * pitch;
  const int tid = threadIdx.x;
  const int64_t p0 = blk * kPrepPts;
  const int fl = tid & 15, rl = tid >> 4;
  double x[NS][2];
#pragma unroll
  for (int j = 0; j < NS; ++j)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int f = 16 * j + fl < d ? 16 * j + fl : d - 1;
      const int64_t p = p0 + rl + 16 * q < n ? p0 + rl + 16 * q : n - 1;
      x[j][q] = X[p * d + f];
    }
  if (tid < kPrepPts) bad[tid] = 0;
  if (tid < d) {
    double c;
    if (ce.part) {
      double w[kMeanFold];
#pragma unroll
      for (int u = 0; u < kMeanFold; ++u) w[u] = ce.part[(int64_t)(u < ce.nblk ? u : ce.nblk - 1) * d + tid];
      c = 0.0;
#pragma unroll
      for (int u = 0; u < kMeanFold; ++u)
        if (u < ce.nblk) c += w[u];
      c /= (double)ce.n;
      if (blockIdx.x == 0) ce.ctr[tid] = c;
    } else {
      c = ce.ctr[tid];
    }
    cm[tid] = c;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    const int f = 16 * j + fl;
    if (f < d) {
      const double s = sc.s[f], c = cm[f];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int r = rl + 16 * q;
        const bool live = p0 + r < n;
        const double v = (x[j][q] - c) * s;
        const double h = f16_round(v);
        const double l = f16_round(v - h);
        if (live && !(__builtin_fabs(v) <= kMaxScaled)) bad[r] = 1;  // every writer writes 1
        const _Float16 h16 = (_Float16)(float)(live ? h : 0.0), l16 = (_Float16)(float)(live ? l : 0.0);
        const _Float16 h2 = (_Float16)(float)(live ? -2.0 * h : 0.0), l2 = (_Float16)(float)(live ? -2.0 * l : 0.0);
        _Float16* const rr = Rr + r * pitch;
        _Float16* const rc = Rc + r * pitch;
        rr[f] = h2;
        rr[d + f] = h2;
        rr[2 * d + f] = l2;
        rc[f] = h16;
        rc[d + f] = l16;
        rc[2 * d + f] = h16;
      }
    }
  }
  __syncthreads();
  if (tid < kPrepPts) {
    const int64_t p = p0 + tid;
    _Float16* const rr = Rr + tid * pitch;
    _Float16* const rc = Rc + tid * pitch;
    double s = 0.0;
    for (int f = 0; f < d; ++f) {
#pragma clang fp contract(off)
      const double t = (double)rc[f] + (double)rc[d + f];
      s += t * t;
    }
    if (bad[tid] || !(s <= kMaxNorm)) s = __builtin_nan("");
    if (nrm) nrm[p] = p < n ? s : 0.0;
    double rem = s;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const double dig = f16_round(rem * (1.0 / (double)kNormScale[q]));  // powers of two: exact
      rem -= dig * (double)kNormScale[q];
      const _Float16 dh = (_Float16)(float)(p < n ? dig : 0.0), ch = (_Float16)(p < n ? kNormScale[q] : 0.f);
      rr[3 * d + q] = dh;
      rr[3 * d + 3 + q] = ch;
      rc[3 * d + q] = ch;
      rc[3 * d + 3 + q] = dh;
    }
    for (int k = 3 * d + 6; k < 32 * KS; ++k) rr[k] = rc[k] = (_Float16)0.f;
  }
  __syncthreads();
  // unit u of the workgroup: point block u / (64 KS), K step, lane
  const int64_t u0 = blk * (kPrepPts / 16) * KS * 64;
  for (int u = tid; u < (kPrepPts / 16) * KS * 64; u += 256) {
    const int lane = u & 63, bk = u >> 6;
    const int blk = bk >= KS ? 1 : 0, ks = bk - blk * KS;
    const int at = (16 * blk + (lane & 15)) * pitch + 32 * ks + 8 * (lane >> 4);
    if (xr) xr[u0 + u] = *(const bf16x8*)(Rr + at);
    if (xc) xc[u0 + u] = *(const bf16x8*)(Rc + at);
  }
}

template <int NS>
__global__ __launch_bounds__(256) void prep_points_f16x3_kernel(PointSet ps, Centre ce, int d, int KS, Scale sc) {
  prep_points_block<NS>(ps, ce, blockIdx.x, d, KS, sc);
}

static size_t prep_points_lds(int KS) { return 2 * (size_t)kPrepPts * (32 * KS + 8) * sizeof(_Float16); }

static hipError_t launch_prep_points(const double* X, const double* ctr, int64_t n, int64_t npad, int d, int KS,
                                     const Scale& sc, void* xr, void* xc, double* nrm, hipStream_t st) {
  static_assert(kPrepPts == 32, "two point blocks per workgroup");
  if (npad % kPrepPts != 0) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)(npad / kPrepPts);
  const size_t lds = prep_points_lds(KS);
  const PointSet ps{X, n, (bf16x8*)xr, (bf16x8*)xc, nrm};
  const Centre ce{const_cast<double*>(ctr), nullptr, 0, 0};
#define GPK_PREP(NS) prep_points_f16x3_kernel<NS><<<grid, 256, lds, st>>>(ps, ce, d, KS, sc)
  switch ((d + 15) / 16) {
    case 1: GPK_PREP(1); break;
    case 2: GPK_PREP(2); break;
    case 3: GPK_PREP(3); break;
    case 4: GPK_PREP(4); break;
    default: GPK_PREP(8); break;
  }
#undef GPK_PREP
  return hipGetLastError();
}

// FP32 point fragments: float4 (blk, q, lane) = f(point 16 blk + lane%16, feature
// 16 q + 4 s + lane/16) for s = 0..3, f = -2 x~ (row side) or x~ (column side).
__global__ void prep_frag_fp32_kernel(const double* __restrict__ X, const double* __restrict__ nrm,
                                      int64_t n, int64_t nblk, int d, int KQ, Scale sc,
                                      f32x4* __restrict__ xr, f32x4* __restrict__ xc,
                                      float* __restrict__ nrm_r, float* __restrict__ nrm_c) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nblk * KQ * 64) return;
  const int lane = (int)(idx & 63);
  const int64_t rest = idx >> 6;
  const int q = (int)(rest % KQ);
  const int64_t blk = rest / KQ;
  const int64_t p = blk * 16 + (lane & 15);
  const int g = lane >> 4;
  f32x4 r, c;
  for (int s = 0; s < 4; ++s) {
    const int f = 16 * q + 4 * s + g;
    float v = 0.f;
    if (p < n && f < d) v = (float)(X[p * d + f] * sc.s[f]);
    r[s] = -2.f * v;
    c[s] = v;
  }
  if (xr) xr[idx] = r;
  if (xc) xc[idx] = c;
  if (q == 0 && g == 0) {
    const float nv = p < n ? (float)nrm[p] : 0.f;
    if (nrm_r) nrm_r[p] = nv;
    if (nrm_c) nrm_c[p] = nv;
  }
}

// Column scales of the mixed form's V fragments.  vmax_partial_kernel: the
// largest |V| of each column over kVParts row ranges (NaN entries are skipped
// here and reach the products through the values themselves); column_exponent:
// scale = 2^e with e = 15 - E, max |V_c| = f 2^E (f in [1/2, 1)), so that the
// scaled column's largest entry lies in [2^14, 2^15), and inv = 2^(-e - 15),
// the factor that takes a partial sum of (kMScale m)(scale V) back to m V.  A zero
// or non-finite column keeps scale 1; e is clamped to [-1022, 1023], which only a
// column whose largest entry lies below 2^-1008 reaches (its scaled entries then stay
// below 2^15 and, down to 2^-1046 relative to that, in FP16's normal range).
constexpr int kVParts = 64;

__device__ __forceinline__ void vmax_partial(const double* __restrict__ V, int64_t ldv, const double* __restrict__ col0,
                                             int64_t n, int c, int q, double* __restrict__ part) {
  __shared__ double red[256];
  const int64_t per = (n + kVParts - 1) / kVParts;
  const int64_t r0 = q * per;
  const int64_t r1 = r0 + per < n ? r0 + per : n;
  const double* src = col0 ? (c == 0 ? col0 : V + (int64_t)(c - 1) * ldv) : V + (int64_t)c * ldv;
  double mx = 0.0;
  for (int64_t b = r0 + threadIdx.x; b < r1; b += 256) mx = fmax(mx, fabs(src[b]));
  red[threadIdx.x] = mx;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[(int64_t)c * kVParts + q] = red[0];
}

__global__ __launch_bounds__(256) void vmax_partial_kernel(const double* __restrict__ V, int64_t ldv,
                                                           const double* __restrict__ col0, int64_t n,
                                                           double* __restrict__ part) {
  vmax_partial(V, ldv, col0, n, blockIdx.y, blockIdx.x, part);
}

__device__ __forceinline__ int column_exponent(double mx) {
  if (!(mx > 0.0 && mx <= 1.7976931348623157e308)) return 0;
  int E = 0;
  (void)frexp(mx, &E);
  const int e = 15 - E;
  return e < -1022 ? -1022 : (e > 1023 ? 1023 : e);  // 2^e and 2^(-e - 15) stay representable
}

__global__ void colmax_final_kernel(const double* __restrict__ part, int t, double* __restrict__ out) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= t) return;
  double mx = 0.0;
  for (int q = 0; q < kVParts; ++q) mx = fmax(mx, part[(int64_t)c * kVParts + q]);
  out[c] = mx;
}

size_t column_absmax_scratch_doubles(int t) { return (size_t)kVParts * (size_t)t; }

hipError_t column_absmax(const double* V, int64_t ldv, int64_t n, int t, double* part, double* out, hipStream_t st) {
  if (!V || !part || !out || t < 1 || n < 1) return hipErrorInvalidValue;
  vmax_partial_kernel<<<dim3(kVParts, (unsigned)t), 256, 0, st>>>(V, ldv, nullptr, n, part);
  colmax_final_kernel<<<(unsigned)((t + 63) / 64), 64, 0, st>>>(part, t, out);
  return hipGetLastError();
}

// Mixed-form V fragments: (chunk, cb, hl, lane) -> 8 FP16 of v' = scale[c] V[b][c],
// b = 32 chunk + vperm(g, j), c = 16 cb + lane%16; hl = 0: hi = RNE16(v'),
// hl = 1: lo = RNE16(v' - hi).  Columns c >= t are zero.  Every wave derives its
// columns' scales from the kVParts maxima (a quarter per lane group), once for the
// `per` chunks it converts; the first chunk's waves store inv.
struct VSet {
  const double* V;
  int64_t ldv;
  const double* col0;
  const double* part;  // column maxima
  double* inv;
  int64_t n, nchunks;
  int t, ntb, per;
  bf16x8* vf;
};

__device__ __forceinline__ void prep_v_block(const VSet& vs, int64_t blk) {
  const double* __restrict__ V = vs.V;
  const double* __restrict__ col0 = vs.col0;
  const double* __restrict__ part = vs.part;
  double* __restrict__ inv = vs.inv;
  bf16x8* __restrict__ vf = vs.vf;
  const int64_t n = vs.n, nchunks = vs.nchunks, ldv = vs.ldv;
  const int t = vs.t, ntb = vs.ntb, per = vs.per;
  const int64_t idx = blk * 256 + threadIdx.x;
  const int lane = (int)(idx & 63);
  const int cb = (int)((idx >> 6) % ntb);
  const int64_t ch0 = (idx >> 6) / ntb * per;  // this wave: chunks ch0 .. ch0 + per - 1 of column block cb
  if (ch0 >= nchunks) return;
  const int64_t ch1 = ch0 + per < nchunks ? ch0 + per : nchunks;
  const int c = 16 * cb + (lane & 15);
  const int g = lane >> 4;
  const int cc = c < t ? c : t - 1;
  const double* const src = col0 ? (cc == 0 ? col0 : V + (int64_t)(cc - 1) * ldv) : V + (int64_t)cc * ldv;
  double pm[kVParts / 4];
#pragma unroll
  for (int q = 0; q < kVParts / 4; ++q) pm[q] = part[(int64_t)cc * kVParts + g * (kVParts / 4) + q];
  double v[8];
  auto load = [&](int64_t ch) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int64_t b = ch * 32 + vperm(g, j);
      v[j] = src[b < n ? b : n - 1];
    }
  };
  load(ch0);
  double mx = 0.0;
#pragma unroll
  for (int q = 0; q < kVParts / 4; ++q) mx = fmax(mx, pm[q]);
  mx = fmax(mx, __shfl_xor(mx, 16, 64));
  mx = fmax(mx, __shfl_xor(mx, 32, 64));
  const int e = column_exponent(mx);
  const double sc = ldexp(1.0, e);
  if (ch0 == 0 && g == 0 && c < t) inv[c] = ldexp(1.0, -e - 15);
  for (int64_t ch = ch0; ch < ch1; ++ch) {
    f16x8 hi, lo;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int64_t b = ch * 32 + vperm(g, j);
      const double x = b < n && c < t ? sc * v[j] : 0.0;
      const double h = f16_round(x);
      hi[j] = (_Float16)(float)h;
      lo[j] = (_Float16)(float)(x - h);
    }
    if (ch + 1 < ch1) load(ch + 1);
    const int64_t rest = ch * ntb + cb;
    vf[(rest * 2 + 0) * 64 + lane] = __builtin_bit_cast(bf16x8, hi);
    vf[(rest * 2 + 1) * 64 + lane] = __builtin_bit_cast(bf16x8, lo);
  }
}

__global__ __launch_bounds__(256) void prep_v_f16x3_kernel(VSet vs) { prep_v_block(vs, blockIdx.x); }

// One product's operands in two launches (three beyond kMeanFold blocks of rows): the
// sums and maxima of X and V, then the fragments of X, of Z (a cross product's rows)
// and of V.  A small product is bound by its launches: n = 2,048, d = 32, t = 9: 33 us
// with one launch per operand and pass (7), 23 so (4).
__global__ __launch_bounds__(256) void prep_reduce_f16x3_kernel(const double* __restrict__ X, int64_t n, int d,
                                                                int64_t rows_per_blk, int nmean,
                                                                double* __restrict__ mpart,
                                                                const double* __restrict__ V, int64_t ldv,
                                                                double* __restrict__ vpart) {
  if ((int)blockIdx.x < nmean) {
    colmean_partial(X, n, d, rows_per_blk, blockIdx.x, mpart);
    return;
  }
  const int b = blockIdx.x - nmean;
  vmax_partial(V, ldv, nullptr, n, b / kVParts, b % kVParts, vpart);
}

template <int NS>
__global__ __launch_bounds__(256) void prep_operands_f16x3_kernel(PointSet px, PointSet pz, int64_t nbx, int64_t nbz,
                                                                  Centre ce, int d, int KS, Scale sc, VSet vs) {
  const int64_t b = blockIdx.x;
  if (b < nbx)
    prep_points_block<NS>(px, ce, b, d, KS, sc);
  else if (b < nbx + nbz)
    prep_points_block<NS>(pz, ce, b - nbx, d, KS, sc);
  else
    prep_v_block(vs, b - nbx - nbz);
}

// FP32 V fragments: (chunk, cb, tile, lane) -> float4 of V[b = 32 chunk + 16 tile + 4g + i]
// [c = 16 cb + lane%16], i = 0..3.
__global__ void prep_v_fp32_kernel(const double* __restrict__ V, int64_t ldv, const double* __restrict__ col0,
                                   int64_t n, int t, int64_t nchunks, int ntb, f32x4* __restrict__ vf) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nchunks * ntb * 2 * 64) return;
  const int lane = (int)(idx & 63);
  const int64_t rest = idx >> 6;  // (ch * ntb + cb) * 2 + tile
  const int tile = (int)(rest & 1);
  const int64_t cbch = rest >> 1;
  const int cb = (int)(cbch % ntb);
  const int64_t ch = cbch / ntb;
  const int c = 16 * cb + (lane & 15);
  const int g = lane >> 4;
  f32x4 o;
  for (int i = 0; i < 4; ++i) {
    const int64_t b = ch * 32 + 16 * tile + 4 * g + i;
    double v = 0.0;
    if (b < n && c < t) v = col0 ? (c == 0 ? col0[b] : V[(int64_t)(c - 1) * ldv + b]) : V[(int64_t)c * ldv + b];
    o[i] = (float)v;
  }
  vf[idx] = o;
}

// ------------------------------------------------------------------ main sweep

struct SweepArgs {
  const void* xr;
  const void* xc;
  const float* nrm_b;
  const float* nrm_a;
  const void* vf;
  double* part;
  int64_t mpad;
  int64_t nchunks;
  int64_t cps;   // chunks per split
  int ntb;       // 16-column blocks in vf
  int tpad;      // columns of the partial buffer
  int t;         // columns that hold a result; the others are not stored
  int f32part;   // cps <= kFlush: each split is one FP32 window, stored exactly as FP32
  int square;    // mask the diagonal (square product)
};

// 16-row blocks per wave: each staged b-stream fragment serves NA tiles and
// each V fragment NA row blocks, as far as 256 registers (two waves per SIMD)
// allow.  n = 65,536 (KS = 13: 40,000), ms, this NA and the next smaller or larger one:
// KS 5 NT 1: 1.82 (2: 1.98); KS 7 NT 1: 2.10 (2: 2.28), NT 4: 3.07 (1: 3.79);
// KS 13 NT 1: 1.36 (4, spilling: 5.66; 1: 1.66), NT 2: 1.74 (2, spilling: 3.59),
// NT 3: 1.85 (2, spilling: 6.41).  With two column blocks and KS <= 5 the kernel fits three
// waves per SIMD (RBF KS 5 NT 2: 1.95 -> 1.84 ms).
template <int KS, int NT>
struct NAOf {
  static constexpr int value = NT == 1 ? (KS <= 7 ? 4 : 2) : (KS <= 7 ? 2 : 1);
  static constexpr int occupancy = NT == 2 && KS <= 5 ? 3 : 2;
};

// partial[(split * tpad + col) * mpad + row .. row + 3] of one 16 x 16 block of sums.
// Columns of the padding are not stored, nor are FP64 zeros: a split of one window is
// an FP32 number (n = 100,003, m = 3,001, t = 33: 302 MB of partials before, 104 now;
// n = 5,001, t = 33: 73 -> 63 us).
__device__ __forceinline__ void store_partial(const SweepArgs& a, int64_t split, int64_t col, int64_t row,
                                              const double* v) {
  if (col >= a.t) return;
  const int64_t o = (split * a.tpad + col) * a.mpad + row;
  if (a.f32part) {
    *(f32x4*)((float*)a.part + o) = f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) a.part[o + i] = v[i];
  }
}

// One 32-point chunk of the b stream staged in LDS: the 2 KS point fragments
// followed by the NT (hi, lo) V fragments, 64 lanes x 16 bytes each.
template <int KS, int NT>
struct ChunkUnits {
  static constexpr int kPoint = 2 * KS * 64;
  static constexpr int kV = 2 * NT * 64;
  static constexpr int kAll = kPoint + kV;
};

template <int KS, int NT, int KIND>
__global__ __launch_bounds__(256, (NAOf<KS, NT>::occupancy)) void sweep_bf16x3_kernel(SweepArgs a) {
  constexpr int NA = NAOf<KS, NT>::value;
  using CU = ChunkUnits<KS, NT>;
  __shared__ bf16x8 stage[2][CU::kAll];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int g = lane >> 4;
  const int64_t ablk0 = ((int64_t)blockIdx.x * 4 + wave) * NA;  // every wave is live: mpad % (64 NA) == 0
  const int cb0 = blockIdx.z * NT;
  const bf16x8* __restrict__ xr = (const bf16x8*)a.xr;
  const bf16x8* __restrict__ xc = (const bf16x8*)a.xc;
  const bf16x8* __restrict__ vf = (const bf16x8*)a.vf;

  bf16x8 A[NA][KS];
#pragma unroll
  for (int ab = 0; ab < NA; ++ab)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) A[ab][ks] = xc[((ablk0 + ab) * KS + ks) * 64 + lane];

  double acc64[NA][NT][4];
  f32x4 acc[NA][NT];
#pragma unroll
  for (int ab = 0; ab < NA; ++ab)
#pragma unroll
    for (int cb = 0; cb < NT; ++cb) {
      acc[ab][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 4; ++i) acc64[ab][cb][i] = 0.0;
    }

  const int64_t c_begin = (int64_t)blockIdx.y * a.cps;
  const int64_t c_end = c_begin + a.cps < a.nchunks ? c_begin + a.cps : a.nchunks;
  const int nch = (int)(c_end - c_begin);
  const int wu = __builtin_amdgcn_readfirstlane(wave);
  // the chunk that holds the points of this wave's first row block
  const int adiag = (int)((((int64_t)blockIdx.x * 4 + wu) * NA >> 1) - c_begin);

  // Copy the next chunk into stage[buf] with direct global-to-LDS loads: the 64-lane
  // units (16 bytes per lane) of the two streams are dealt to the waves in turn (unit
  // j to wave j mod 4), so source and LDS slot of every load are fixed up to the wave
  // index, which is held in a scalar register; no registers hold the data in flight.
  // Completion is awaited and published by the barrier that ends the iteration.  n = 262,144, d = 48, t = 16: 31.2 ms through registers with
  // per-thread addresses, 29.3 so, 28.9 with the diagonal below as a scalar branch;
  // two chunks per barrier: the same.
  const bf16x8* px = xr + c_begin * (2 * KS * 64) + tid;
  const bf16x8* pv = vf + (c_begin * a.ntb + cb0) * 2 * 64 + tid;
  auto load_stream = [&](const bf16x8* src, int units, int first, int buf) {
#pragma unroll
    for (int r = 0; r < (units + 3) / 4; ++r) {
      const int j = wu + 4 * r;
      if (j < units)
        __builtin_amdgcn_global_load_lds((const void*)(src + 256 * r),
                                         (__attribute__((address_space(3))) void*)&stage[buf][first + 64 * j], 16, 0,
                                         0);
    }
  };
  auto fetch = [&](int ch, int buf) {
    if (ch < nch) {
      load_stream(px, 2 * KS, 0, buf);
      load_stream(pv, 2 * NT, CU::kPoint, buf);
    }
    px += 2 * KS * 64;
    pv += (int64_t)a.ntb * 2 * 64;
  };
  fetch(0, 0);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  int cur = 0;
  for (int ch = 0; ch < nch; ++ch, cur ^= 1) {
    const bool more = ch + 1 < nch;
    bf16x8 B0[KS], B1[KS], VH[NT], VL[NT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      B0[ks] = stage[cur][ks * 64 + lane];
      B1[ks] = stage[cur][(KS + ks) * 64 + lane];
    }
#pragma unroll
    for (int cb = 0; cb < NT; ++cb) {
      VH[cb] = stage[cur][CU::kPoint + (2 * cb) * 64 + lane];
      VL[cb] = stage[cur][CU::kPoint + (2 * cb + 1) * 64 + lane];
    }
    fetch(ch + 1, cur ^ 1);
#pragma unroll
    for (int ab = 0; ab < NA; ++ab) {
      f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        s0 = mfma_dist(B0[ks], A[ab][ks], s0);
        s1 = mfma_dist(B1[ks], A[ab][ks], s1);
      }
      f32x8 mv;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        mv[i] = profile_scaled<KIND>(s0[i]);
        mv[4 + i] = profile_scaled<KIND>(s1[i]);
      }
      if (a.square) {
        if (NA == 1 ? adiag == ch : adiag + (ab >> 1) == ch) {
          const int off = (NA == 1 ? (wu & 1) : (ab & 1)) ? 4 : 0;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if ((lane & 15) == 4 * g + i) mv[off + i] = 0.f;
        }
      }
      bf16x8 H, L;
      split_f16x8(mv, H, L);
#pragma unroll
      for (int cb = 0; cb < NT; ++cb) {
        acc[ab][cb] = mfma_val(H, VH[cb], acc[ab][cb]);
        acc[ab][cb] = mfma_val(H, VL[cb], acc[ab][cb]);
        acc[ab][cb] = mfma_val(L, VH[cb], acc[ab][cb]);
      }
    }
    if (((ch + 1) % kFlush) == 0 || !more) {
#pragma unroll
      for (int ab = 0; ab < NA; ++ab)
#pragma unroll
        for (int cb = 0; cb < NT; ++cb) {
#pragma unroll
          for (int i = 0; i < 4; ++i) acc64[ab][cb][i] += (double)acc[ab][cb][i];
          acc[ab][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  }
#pragma unroll
  for (int ab = 0; ab < NA; ++ab)
#pragma unroll
    for (int cb = 0; cb < NT; ++cb)
      store_partial(a, blockIdx.y, (int64_t)(cb0 + cb) * 16 + (lane & 15), (ablk0 + ab) * 16 + 4 * g, acc64[ab][cb]);
}

// ------------------------------------------------------------------ wide cross sweep
//
// The prediction product K(Z, X) [alpha | R] has few query rows (a request
// batch) and many columns (1 + k_c).  The sweep above evaluates each kernel
// entry once per 64-column group; here a workgroup owns 64 query rows and all
// columns of one chunk split.  Per 32-point chunk, wave w evaluates the
// distances and the profile of row block w (16 rows) into an LDS tile (FP16
// hi / lo, two buffers so that one barrier per chunk suffices); then every
// wave multiplies the four row blocks' tiles by its own column blocks (cb = w,
// w + 4, ...), and of the column blocks left over (257 columns: one) its own row
// block's tile, so that the waves do the same work: 51 instead of 60 MFMA in the
// busiest one.  Both operand streams run ahead in registers: the point fragments
// of chunk c + 1 are loaded during chunk c - 1 and written to LDS at the top of
// chunk c, and each wave's V fragments of chunk c + 1 are loaded during chunk c
// into the other of two register sets.  FP32 windows of kFlush chunks are
// added into the split's FP64 partials (this workgroup owns those slots) in the
// same order as the sweep above, so each output row's sums depend on n only, not
// on the batch; a split of one window stores it as FP32, which is exact and halves
// the partials' traffic.  Workgroups are numbered so that the row groups of
// one split run back to back on one XCD and share the chunk data in its L2.
//
// A batch of 1,200 rows (n = 262,144, d = 48, 257 columns) is bound by the matrix
// cores (busy 48%, about what a mix of MFMA and VALU work reaches here) and the
// 2 x 313 MB of its partials: mean and variance 696 -> 648 us; 24 rows are bound by
// the streams: 89 -> 86 us (354 MB: 74 us at the copy rate); with few columns
// the leftover rule spreads them over the waves: 41 columns 429 -> 244 us, one
// column 423 -> 189 us.  Tried: direct global-to-LDS loads for the points (the
// compiler then waits for every load in flight at each LDS read and barrier: 718 us
// with two register sets, 654 with one and three workgroups per CU, but 100 us at 24 rows).
constexpr int kWideBlocks = 20;  // column blocks: 320 columns >= 1 + 256

struct WideArgs {
  const void* xr;  // b stream (training points)
  const void* xc;  // query-row fragments
  const void* vf;  // V fragments, vstride 16-column blocks per chunk
  double* part;    // [split][tpad][mpad], FP64, or FP32 when f32part
  int64_t m, mpad, nchunks, cps, nsplit;
  int t, ntb, vstride, tpad, rgroups;  // columns, column blocks
  int f32part;  // cps <= kFlush: each split is one FP32 window, stored exactly as FP32
};

template <int KS, int FULL, int REST, int KIND>
__global__ __launch_bounds__(256, 2) void wide_cross_bf16x3_kernel(WideArgs a) {
  constexpr int kPoint = 2 * KS * 64;  // 16-byte units of one chunk's point fragments
  __shared__ bf16x8 stage[2][kPoint];
  __shared__ bf16x8 tile[2][4][2][64];  // [parity][row block][hi / lo][lane]
  // hardware workgroup i runs on XCD i % 8; the j-th workgroup an XCD receives
  // (j = i / 8) takes row group j % R of split 8 (j / R) + i % 8
  const int64_t hw = blockIdx.x;
  const int64_t j8 = hw >> 3;
  const int rg = (int)(j8 % a.rgroups);
  const int64_t split = (j8 / a.rgroups) * 8 + (hw & 7);
  if (split >= a.nsplit) return;  // whole workgroup, before any barrier
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wu = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t ablk = (int64_t)rg * 4 + wu;  // this wave's row block (16 rows)
  const bool live = ablk * 16 < a.m;          // it holds a query row
  const bool live2 = (int64_t)rg * 64 + 32 < a.m;  // so does one of the last two row blocks
  const bf16x8* __restrict__ xc = (const bf16x8*)a.xc;
  bf16x8 A[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) A[ks] = xc[(ablk * KS + ks) * 64 + lane];
  f32x4 acc[4][FULL > 0 ? FULL : 1], accr[REST > 0 ? REST : 1];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
#pragma unroll
    for (int jb = 0; jb < FULL; ++jb) acc[rb][jb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < REST; ++j) accr[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int64_t c_begin = split * a.cps;
  const int64_t c_end = c_begin + a.cps < a.nchunks ? c_begin + a.cps : a.nchunks;
  const int nch = (int)(c_end - c_begin);  // >= 1

  // Loads are unconditional (units, blocks and chunks beyond the last repeat the last
  // one), so that the number in flight is the same on every path and a wait covers
  // only what its use needs.
  constexpr int kPer = (2 * KS + 3) / 4;
  const bf16x8* const xr = (const bf16x8*)a.xr + c_begin * kPoint + lane;
  bf16x8 pre[kPer];
  auto fetch = [&](int ch) {  // the points of chunk ch, 64-lane unit j by wave j mod 4
    const bf16x8* const src = xr + (int64_t)(ch < nch ? ch : nch - 1) * kPoint;
#pragma unroll
    for (int r = 0; r < kPer; ++r) pre[r] = src[64 * (wu + 4 * r < 2 * KS ? wu + 4 * r : 2 * KS - 1)];
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int r = 0; r < kPer; ++r)
      if (wu + 4 * r < 2 * KS) stage[buf][64 * (wu + 4 * r) + lane] = pre[r];
  };
  const int64_t vstep = (int64_t)a.vstride * 2 * 64;
  const bf16x8* const vf = (const bf16x8*)a.vf + c_begin * vstep;
  struct VFrag {
    bf16x8 f[FULL + REST][2];
  };
  auto vload = [&](int ch, VFrag& v) {
    const bf16x8* const src = vf + (int64_t)(ch < nch ? ch : nch - 1) * vstep;
#pragma unroll
    for (int j = 0; j < FULL + REST; ++j) {
      int cb = j < FULL ? wu + 4 * j : 3 * FULL + j;
      cb = cb < a.ntb ? cb : a.ntb - 1;
      v.f[j][0] = (src + (int64_t)cb * 128)[lane];
      v.f[j][1] = (src + (int64_t)cb * 128 + 64)[lane];
    }
  };
  // one column block's sums of row block rb into the partials
  bool first_window = true;
  auto put = [&](int cb, int rb, const f32x4& v) {
    const int64_t col = (int64_t)cb * 16 + (lane & 15);
    if (col >= a.t) return;
    const int64_t o = (split * a.tpad + col) * a.mpad + (int64_t)rg * 64 + 16 * rb + 4 * (lane >> 4);
    if (a.f32part) {
      *(f32x4*)((float*)a.part + o) = v;
    } else {
      double* dst = a.part + o;
      double old[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) old[i] = first_window ? 0.0 : dst[i];
#pragma unroll
      for (int i = 0; i < 4; ++i) dst[i] = old[i] + (double)v[i];
    }
  };
  auto flush = [&]() {
#pragma unroll
    for (int jb = 0; jb < FULL; ++jb)
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) {
        put(wu + 4 * jb, rb, acc[rb][jb]);
        acc[rb][jb] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
    for (int j = 0; j < REST; ++j) {
      put(4 * FULL + j, wu, accr[j]);
      accr[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    first_window = false;
  };

  auto chunk = [&](int ch, const VFrag& V, VFrag& Vn) {
    const int cur = ch & 1;
    // stage[cur ^ 1] was last read in phase A of the previous chunk
    stash(cur ^ 1);
    fetch(ch + 2);
    vload(ch + 1, Vn);
    // phase A: this wave's row block against the chunk
    bf16x8 H, L;
    if (live) {
      f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        s0 = mfma_dist(stage[cur][ks * 64 + lane], A[ks], s0);
        s1 = mfma_dist(stage[cur][(KS + ks) * 64 + lane], A[ks], s1);
      }
      f32x8 mv;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        mv[i] = profile_scaled<KIND>(s0[i]);
        mv[4 + i] = profile_scaled<KIND>(s1[i]);
      }
      split_f16x8(mv, H, L);
      tile[cur][wu][0][lane] = H;
      tile[cur][wu][1][lane] = L;
    }
    // the four tiles of this chunk, and the next chunk's points, are in LDS
    __syncthreads();
    // phase B: the four row blocks against this wave's column blocks, two at a time
#pragma unroll
    for (int rp = 0; rp < 4; rp += 2) {
      if (rp == 0 || live2) {
        bf16x8 T[2][2];
        if (FULL > 0) {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            T[i][0] = tile[cur][rp + i][0][lane];
            T[i][1] = tile[cur][rp + i][1][lane];
          }
        }
#pragma unroll
        for (int jb = 0; jb < FULL; ++jb) {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            acc[rp + i][jb] = mfma_val(T[i][0], V.f[jb][0], acc[rp + i][jb]);
            acc[rp + i][jb] = mfma_val(T[i][0], V.f[jb][1], acc[rp + i][jb]);
            acc[rp + i][jb] = mfma_val(T[i][1], V.f[jb][0], acc[rp + i][jb]);
          }
        }
      }
    }
    if (live) {
#pragma unroll
      for (int j = 0; j < REST; ++j) {
        accr[j] = mfma_val(H, V.f[FULL + j][0], accr[j]);
        accr[j] = mfma_val(H, V.f[FULL + j][1], accr[j]);
        accr[j] = mfma_val(L, V.f[FULL + j][0], accr[j]);
      }
    }
    if (((ch + 1) % kFlush) == 0 || ch + 1 == nch) flush();
  };
  VFrag V0, V1;
  fetch(0);
  stash(0);
  fetch(1);
  vload(0, V0);
  __syncthreads();
  for (int ch = 0; ch < nch; ch += 2) {
    chunk(ch, V0, V1);
    if (ch + 1 < nch) chunk(ch + 1, V1, V0);
  }
}

// 16-row blocks per wave of the FP32 form, one or two.  An MFMA of this form takes twice
// the cycles for an eighth of the flops, so that a fragment's LDS read costs little
// beside it: with two blocks the work itself gets pair_gain_f32 (per mille) faster, more
// under RBF, whose shorter profile leaves the reads exposed; -1: not at all (n = 65,536,
// Matern: KQ 3 NT 1 5.43 ms with one, 5.56 with two) or two blocks spill.  Measured
// where both fill the CUs, one / two blocks, ms: RBF n = 110,000, d = 48, t = 1 14.9 / 12.3, t
// = 17 17.7 / 16.4; n = 30,000, d = 48, t = 40 1.68 / 1.50, d = 100, t = 20 2.72 / 2.35; Matern n =
// 30,000, d = 48, t = 64 2.02 / 1.97, d = 21, t = 40 1.55 / 1.54, d = 100, t = 1 2.35 / 2.22.
//
// But half as many workgroups of twice the work may leave CUs idle: with w of them the
// busiest CU does 2 ceil(w / 256) halves against ceil(2 w / 256).  That ratio, where it is above
// one, is what two blocks cost (Matern, d = 5, t = 40: n = 20,000, w = 1,106, 10 against 9: 0.578 /
// 0.644 ms; RBF, d = 21, t = 17: n = 2,500, w = 800, 8 against 7: 28.7 / 30.3 us), so two
// are taken where the gain makes up for it.  A row's sums are the same with either.
constexpr int pair_gain_f32(int kq, int nt, int kind) {
  if (kq > 4) return nt > 2 ? -1 : (kind == GP_RBF ? 112 : 60);
  if (kind == GP_RBF) return nt > 2 ? 112 : 67;
  return nt > 2 ? 10 : -1;
}

static int na_f32(int kq, int nt, int kind, int64_t mpad, int64_t nsplit, int64_t groups) {
  const int gain = pair_gain_f32(kq, nt, kind);
  const int64_t w = mpad / 128 * nsplit * groups;
  return gain >= 0 && 2 * ((w + 255) / 256) * 1000 <= (2 * w + 255) / 256 * (1000 + gain) ? 2 : 1;
}

// The FP32 form: distances and M V on v_mfma_f32_16x16x4, bound by them (32 cycles
// each: at KQ = 2, NT = 3 40 per 16 x 32 tile) and the profile's VALU work, which adds
// to them.  Staged as in the mixed form (the norms of the b stream through registers,
// one chunk ahead): with every wave loading its fragments from global memory a
// chunk's loads were awaited before its compute.  K(Z, X) V at n = 100,003, m =
// 3,001, d = 21, t = 33, RBF: 0.62 -> 0.49 ms with FP32 partials; n = 65,536, d =
// 64, t = 50: 11.8 -> 9.5 ms.
template <int KQ, int NT, int KIND, int NA>
__global__ __launch_bounds__(256, 2) void sweep_fp32_kernel(SweepArgs a) {
  constexpr int kPoint = 2 * KQ * 64, kAll = kPoint + 2 * NT * 64;
  __shared__ f32x4 stage[2][kAll];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wu = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4;
  const int64_t ablk0 = ((int64_t)blockIdx.x * 4 + wu) * NA;  // every wave is live: mpad % (64 NA) == 0
  const int cb0 = blockIdx.z * NT;
  const f32x4* __restrict__ xc = (const f32x4*)a.xc;

  f32x4 A[NA][KQ];
  float na[NA];
#pragma unroll
  for (int ab = 0; ab < NA; ++ab) {
#pragma unroll
    for (int q = 0; q < KQ; ++q) A[ab][q] = xc[((ablk0 + ab) * KQ + q) * 64 + lane];
    na[ab] = a.nrm_a[(ablk0 + ab) * 16 + (lane & 15)];
  }
  double acc64[NA][NT][4];
  f32x4 acc[NA][NT];
#pragma unroll
  for (int ab = 0; ab < NA; ++ab)
#pragma unroll
    for (int cb = 0; cb < NT; ++cb) {
      acc[ab][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 4; ++i) acc64[ab][cb][i] = 0.0;
    }

  const int64_t c_begin = (int64_t)blockIdx.y * a.cps;
  const int64_t c_end = c_begin + a.cps < a.nchunks ? c_begin + a.cps : a.nchunks;
  const int nch = (int)(c_end - c_begin);
  const int adiag = (int)((ablk0 >> 1) - c_begin);  // the chunk that holds the points of this wave's first row block

  const f32x4* px = (const f32x4*)a.xr + c_begin * kPoint + tid;
  const f32x4* pv = (const f32x4*)a.vf + (c_begin * a.ntb + cb0) * 2 * 64 + tid;
  const float* pn = a.nrm_b + c_begin * 32 + 4 * g;
  f32x4 nb0 = {0.f, 0.f, 0.f, 0.f}, nb1 = {0.f, 0.f, 0.f, 0.f};
  auto load_stream = [&](const f32x4* src, int units, int first, int buf) {
#pragma unroll
    for (int r = 0; r < (units + 3) / 4; ++r) {
      const int j = wu + 4 * r;
      if (j < units)
        __builtin_amdgcn_global_load_lds((const void*)(src + 256 * r),
                                         (__attribute__((address_space(3))) void*)&stage[buf][first + 64 * j], 16, 0,
                                         0);
    }
  };
  auto fetch = [&](int ch, int buf) {
    if (ch < nch) {
      nb0 = *(const f32x4*)pn;
      nb1 = *(const f32x4*)(pn + 16);
      load_stream(px, 2 * KQ, 0, buf);
      load_stream(pv, 2 * NT, kPoint, buf);
    }
    px += kPoint;
    pv += (int64_t)a.ntb * 2 * 64;
    pn += 32;
  };
  fetch(0, 0);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  int cur = 0;
  for (int ch = 0; ch < nch; ++ch, cur ^= 1) {
    const bool more = ch + 1 < nch;
    f32x4 B0[KQ], B1[KQ], V0[NT], V1[NT];
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
      B0[q] = stage[cur][q * 64 + lane];
      B1[q] = stage[cur][(KQ + q) * 64 + lane];
    }
#pragma unroll
    for (int cb = 0; cb < NT; ++cb) {
      V0[cb] = stage[cur][kPoint + (2 * cb) * 64 + lane];
      V1[cb] = stage[cur][kPoint + (2 * cb + 1) * 64 + lane];
    }
    const f32x4 n0 = nb0, n1 = nb1;
    fetch(ch + 1, cur ^ 1);
#pragma unroll
    for (int ab = 0; ab < NA; ++ab) {
      f32x4 s0 = n0 + na[ab];
      f32x4 s1 = n1 + na[ab];
#pragma unroll
      for (int q = 0; q < KQ; ++q)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(B0[q][s], A[ab][q][s], s0, 0, 0, 0);
          s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(B1[q][s], A[ab][q][s], s1, 0, 0, 0);
        }
      f32x4 m0, m1;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        m0[i] = profile<KIND, true>(s0[i]);
        m1[i] = profile<KIND, true>(s1[i]);
      }
      if (a.square) {
        if (NA == 1 ? adiag == ch : adiag + (ab >> 1) == ch) {
          f32x4& md = (NA == 1 ? (wu & 1) : (ab & 1)) ? m1 : m0;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if ((lane & 15) == 4 * g + i) md[i] = 0.f;
        }
      }
#pragma unroll
      for (int cb = 0; cb < NT; ++cb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[ab][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(m0[i], V0[cb][i], acc[ab][cb], 0, 0, 0);
          acc[ab][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(m1[i], V1[cb][i], acc[ab][cb], 0, 0, 0);
        }
    }
    if (((ch + 1) % kFlush) == 0 || !more) {
#pragma unroll
      for (int ab = 0; ab < NA; ++ab)
#pragma unroll
        for (int cb = 0; cb < NT; ++cb) {
#pragma unroll
          for (int i = 0; i < 4; ++i) acc64[ab][cb][i] += (double)acc[ab][cb][i];
          acc[ab][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  }
#pragma unroll
  for (int ab = 0; ab < NA; ++ab)
#pragma unroll
    for (int cb = 0; cb < NT; ++cb)
      store_partial(a, blockIdx.y, (int64_t)(cb0 + cb) * 16 + (lane & 15), (ablk0 + ab) * 16 + 4 * g, acc64[ab][cb]);
}

// out[c*ldo + r] = s_f * inv[c] * sum_split part + (square ? (s_f + sigma^2) V[c*ldv + r] : 0)
// (inv: the mixed form's column factors, a power of two; null for the FP32 form).
// grid = (row blocks, columns); dot (nullable): dot[b t + c] = sum over the block's
// rows of V out, added as in coldot_partial_kernel.
// Bound by HBM where there is one split (n = 917,504, t = 16: 352 MB in 117 us; 75 us with
// one value in flight per thread and more waves, which many splits are slower with), by the
// partials' reads where there are many.
template <typename T>
__global__ __launch_bounds__(256) void kmm_epilogue_kernel(const T* __restrict__ part, int64_t nsplit, int tpad,
                                                           int64_t mpad, int64_t m, int t, double sf, double diag,
                                                           const double* __restrict__ inv, const double* __restrict__ V,
                                                           int64_t ldv, double* __restrict__ out, int64_t ldo,
                                                           int64_t rows_per_blk, double* __restrict__ dot) {
  __shared__ double sh[4];
  const int64_t c = blockIdx.y;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_blk;
  const int64_t r1 = r0 + rows_per_blk < m ? r0 + rows_per_blk : m;
  double acc = 0.0;
  for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) {
    const double vr = V ? V[c * ldv + r] : 0.0;
    double s = 0.0;
    const T* src = part + c * mpad + r;
    const int64_t step = (int64_t)tpad * mpad;
    int64_t sp = 0;
    for (; sp + 16 <= nsplit; sp += 16, src += 16 * step) {  // in split order, 16 loads in flight
      T v[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) v[j] = src[j * step];
#pragma unroll
      for (int j = 0; j < 16; ++j) s += (double)v[j];
    }
    for (; sp + 4 <= nsplit; sp += 4, src += 4 * step) {
      T v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = src[j * step];
#pragma unroll
      for (int j = 0; j < 4; ++j) s += (double)v[j];
    }
    for (; sp < nsplit; ++sp, src += step) s += (double)src[0];
    if (inv) s *= inv[c];
    double o = sf * s;
    if (V) o += diag * vr;
    out[c * ldo + r] = o;
    acc += vr * o;
  }
  if (dot) {
    const double b = block_sum(acc, sh);
    if (threadIdx.x == 0) dot[(int64_t)blockIdx.x * t + c] = b;
  }
}

// The split sum of the wide sweep: a workgroup takes one column and 64 rows,
// wave k adds the splits k, k + 4, ... in split order, and the four sums are
// then added in wave order, so the order depends on n alone.
template <typename T>
__global__ __launch_bounds__(256) void wide_epilogue_kernel(const T* __restrict__ part, int64_t nsplit, int tpad,
                                                            int64_t mpad, int64_t m, double sf,
                                                            const double* __restrict__ inv,
                                                            double* __restrict__ out, int64_t ldo) {
  __shared__ double red[4][64];
  const int r = threadIdx.x & 63;
  const int k = threadIdx.x >> 6;
  const int64_t q = (int64_t)blockIdx.x * 64 + r;
  const int64_t c = blockIdx.y;
  double s = 0.0;
  if (q < m) {
    // splits k, k + 4, ... added in that order; eight loads in flight per batch
    const int64_t step = 4 * (int64_t)tpad * mpad;
    const T* src = part + ((int64_t)k * tpad + c) * mpad + q;
    int64_t sp = k;
    for (; sp + 28 < nsplit; sp += 32, src += 8 * step) {
      T v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = src[j * step];
#pragma unroll
      for (int j = 0; j < 8; ++j) s += (double)v[j];
    }
    for (; sp < nsplit; sp += 4, src += step) s += (double)src[0];
  }
  red[k][r] = s;
  __syncthreads();
  if (k == 0 && q < m) out[c * ldo + q] = sf * ((((red[0][r] + red[1][r]) + red[2][r]) + red[3][r]) * inv[c]);
}

// ------------------------------------------------------------------ host side

// Optional timing of the tile sweeps: HIP events recorded on the sweep's own
// stream around each launch, with the launch's nominal flops 2 m n (d + t).
namespace {
struct SweepTiming {
  std::mutex mu;
  bool on = false;
  struct Rec {
    hipEvent_t a, b;
    double flops;
    int64_t n, m;
    int t;
  };
  std::vector<Rec> recs;
};
SweepTiming& timing() {
  static SweepTiming t;
  return t;
}
}  // namespace

void profile_enable(bool on) {
  std::lock_guard<std::mutex> g(timing().mu);
  timing().on = on;
}

int profile_records(int64_t cap, int64_t* n, int64_t* m, int* t, double* ms, int64_t* count) {
  std::lock_guard<std::mutex> g(timing().mu);
  int64_t k = 0;
  for (auto& r : timing().recs) {
    if (k >= cap) break;
    if (hipEventSynchronize(r.b) != hipSuccess) return -1;
    float e = 0.f;
    if (hipEventElapsedTime(&e, r.a, r.b) != hipSuccess) return -1;
    n[k] = r.n;
    m[k] = r.m;
    t[k] = r.t;
    ms[k] = e;
    ++k;
  }
  *count = k;
  return 0;
}

int profile_read(int64_t* launches, double* total_ms, double* flops, bool reset) {
  std::lock_guard<std::mutex> g(timing().mu);
  int64_t n = 0;
  double ms = 0.0, fl = 0.0;
  for (auto& r : timing().recs) {
    if (hipEventSynchronize(r.b) != hipSuccess) return -1;
    float e = 0.f;
    if (hipEventElapsedTime(&e, r.a, r.b) != hipSuccess) return -1;
    ms += e;
    fl += r.flops;
    ++n;
  }
  if (reset) {
    for (auto& r : timing().recs) {
      (void)hipEventDestroy(r.a);
      (void)hipEventDestroy(r.b);
    }
    timing().recs.clear();
  }
  *launches = n;
  *total_ms = ms;
  *flops = fl;
  return 0;
}

static int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }
static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

int kmm_ksteps(int precision, int d) {
  if (precision == GP_PREC_FP64) return d <= kF64MaxD ? 1 : -1;
  if (precision == GP_PREC_BF16X3) {
    const int need = (3 * d + 6 + 31) / 32;
    static const int kAvail[] = {2, 4, 5, 7, 13};  // the instantiated sweeps
    for (int k : kAvail)
      if (k >= need) return k;
    return -1;
  }
  const int need = (d + 15) / 16;
  static const int kAvail32[] = {1, 2, 3, 4, 8};  // the instantiated sweeps
  for (int k : kAvail32)
    if (k >= need) return k;
  return -1;
}

// Column blocks handled per launch (grid.z groups the rest).
static int nt_launch(int ntb) { return ntb >= 4 ? 4 : ntb; }
static int na_of(int ks, int nt) {  // NAOf of the launched kernel
  return nt == 1 ? (ks <= 7 ? 4 : 2) : (ks <= 7 ? 2 : 1);
}

// 16-row blocks per wave that the split rule counts with: it fixes the FP32 windows
// and the order of the sums, which stay the same whatever a kernel's registers hold.
static int na_of_split(int ks, int nt, bool mixed) { return nt == 1 ? 4 : nt == 2 || (mixed && ks <= 5) ? 2 : 1; }

struct SplitChoice {
  int nt, groups, tpad;
  int64_t cps, nsplit;
};

static SplitChoice choose_split(int64_t npad, int64_t mpad, int ntb, bool row_independent, int ks, bool mixed) {
  SplitChoice s;
  s.nt = nt_launch(ntb);
  s.groups = (ntb + s.nt - 1) / s.nt;
  s.tpad = s.groups * s.nt * 16;
  const int64_t nchunks = npad / 32;
  if (row_independent) {
    // depends on n only: each output row sees the same chunk boundaries whatever m is
    s.cps = std::max<int64_t>(8, (nchunks + 255) / 256);
  } else {
    const int64_t row_wgs = mpad / (64 * na_of_split(ks, s.nt, mixed)) * s.groups;
    const int64_t want = std::max<int64_t>(1, (2048 + row_wgs - 1) / row_wgs);
    s.cps = std::max<int64_t>(2, (nchunks + want - 1) / want);
  }
  s.nsplit = (nchunks + s.cps - 1) / s.cps;
  return s;
}

static size_t part_bytes_max(int64_t npad, int64_t mpad, int ntb, bool row_independent, int ks, bool mixed) {
  size_t best = 0;
  for (int nb = 1; nb <= ntb; ++nb) {
    const SplitChoice s = choose_split(npad, mpad, nb, row_independent, ks, mixed);
    best = std::max(best, (size_t)s.nsplit * s.tpad * mpad * sizeof(double));
  }
  return best;
}

// V region: [fragments | inv (tpad) | column-max partials (kVParts tpad)].
static size_t vfrag_core_bytes(int64_t n, int ntb_alloc) {
  return align256((size_t)round_up(n, 32) * ntb_alloc * 64 + 64);
}

size_t kmm_vfrag_bytes(int64_t n, int t) {
  const int ntb0 = (t + 15) / 16;
  const int ntb = (ntb0 + nt_launch(ntb0) - 1) / nt_launch(ntb0) * nt_launch(ntb0);
  return vfrag_core_bytes(n, ntb) + align256((size_t)ntb * 16 * 8) + align256((size_t)kVParts * ntb * 16 * 8);
}

static void carve_vfrag(KmmPlan& p, char* c) {
  const int ntb_alloc = (p.ntb + nt_launch(p.ntb) - 1) / nt_launch(p.ntb) * nt_launch(p.ntb);
  const int tpad = ntb_alloc * 16;
  p.vf = c;
  c += vfrag_core_bytes(p.n, ntb_alloc);
  p.vinv = (double*)c;  c += align256((size_t)tpad * 8);
  p.vpart = (double*)c;
}

size_t kmm_plan_bytes(int precision, int d, int64_t n, int64_t m, bool square, int tmax) {
  const int ks = kmm_ksteps(precision, d);
  if (ks < 0) return 0;
  if (precision == GP_PREC_FP64)
    return align256((size_t)d * 8) + align256((size_t)n * 8) + align256(f64_split(n, square ? n : m, square, tmax).bytes) +
           256;
  const int64_t npad = round_up(n, 32);
  const int64_t mrows = square ? n : m;
  const int64_t mpad = round_up(mrows, 256);
  const int64_t bpad = std::max(npad, mpad);  // the square case prepares mpad rows of X
  const int ntb0 = (tmax + 15) / 16;
  size_t b = 0;
  b += align256((size_t)bpad * ks * 64);           // xr
  b += align256((size_t)mpad * ks * 64);           // xc
  b += align256((size_t)bpad * 4);                 // nrm_b
  b += align256((size_t)mpad * 4);                 // nrm_a
  b += align256((size_t)bpad * 8);                 // nrm64
  b += align256((size_t)d * 8);                    // ctr
  b += align256(colmean_scratch_doubles(n, d) * 8);  // column-mean partials
  b += kmm_vfrag_bytes(n, tmax);                   // vf, column scales
  b += align256(part_bytes_max(npad, mpad, ntb0, !square, ks, precision == GP_PREC_BF16X3));  // partials
  return b;
}

bool kmm_plan_init(KmmPlan& p, const gp_kernel* kern, int precision, int64_t n, int64_t m,
                   bool square, int tmax, void* ws, size_t ws_bytes) {
  const size_t need = kmm_plan_bytes(precision, kern->d, n, m, square, tmax);
  if (need == 0 || ws == nullptr || ws_bytes < need) return false;
  p.precision = precision;
  p.kind = kern->kind;
  p.d = kern->d;
  p.square = square;
  p.n = n;
  p.m = square ? n : m;
  p.npad = round_up(n, 32);
  p.mpad = round_up(p.m, 256);
  p.nchunks = p.npad / 32;
  p.ks = kmm_ksteps(precision, kern->d);
  p.tmax = tmax;
  p.ntb = (tmax + 15) / 16;
  p.sf = kern->outputscale;
  p.noise = kern->noise;
  if (precision == GP_PREC_FP64) {
    char* c = (char*)ws;
    p.sc64 = (double*)c;  c += align256((size_t)p.d * 8);
    p.nb64 = (double*)c;  c += align256((size_t)n * 8);
    p.part = (double*)c;
    p.f64 = f64_split(n, p.m, square, tmax);
    return true;
  }
  const int64_t bpad = std::max(p.npad, p.mpad);
  char* c = (char*)ws;
  p.xr = c;  c += align256((size_t)bpad * p.ks * 64);
  p.xc = c;  c += align256((size_t)p.mpad * p.ks * 64);
  p.nrm_b = (float*)c;  c += align256((size_t)bpad * 4);
  p.nrm_a = (float*)c;  c += align256((size_t)p.mpad * 4);
  p.nrm64 = (double*)c; c += align256((size_t)bpad * 8);
  p.ctr = (double*)c;   c += align256((size_t)p.d * 8);
  p.cpart = (double*)c; c += align256(colmean_scratch_doubles(n, p.d) * 8);
  carve_vfrag(p, c);
  c += kmm_vfrag_bytes(n, tmax);
  p.part = (double*)c;
  return true;
}

// Model buffer: [b-stream fragments | b norms (FP32) | V fragments | centre (d) | column-mean and FP64 norm
// scratch of the prepare step].
size_t kmm_model_bytes(int precision, int d, int64_t n, int tmax) {
  if (precision == GP_PREC_FP64) return 0;  // prediction models use the matrix-core forms
  const int ks = kmm_ksteps(precision, d);
  if (ks < 0) return 0;
  const int64_t npad = round_up(n, 32);
  return align256((size_t)npad * ks * 64) + align256((size_t)npad * 4) + kmm_vfrag_bytes(n, tmax) +
         align256((size_t)d * 8) + align256(colmean_scratch_doubles(n, d) * 8) + align256((size_t)npad * 8);
}

// Query workspace: [row fragments | row norms (FP32) | FP64 norm scratch | partials].
size_t kmm_query_bytes(int precision, int d, int64_t n, int64_t m, int tmax) {
  if (precision == GP_PREC_FP64) return 0;
  const int ks = kmm_ksteps(precision, d);
  if (ks < 0) return 0;
  const int64_t npad = round_up(n, 32);
  const int64_t mpad = round_up(m, 256);
  const int ntb = (tmax + 15) / 16;
  return align256((size_t)mpad * ks * 64) + align256((size_t)mpad * 4) + align256((size_t)mpad * 8) +
         align256(part_bytes_max(npad, mpad, ntb, true, ks, precision == GP_PREC_BF16X3));
}

bool kmm_plan_model(KmmPlan& p, const gp_kernel* kern, int precision, int64_t n, int64_t m, int tmax, void* model,
                    size_t model_bytes, void* ws, size_t ws_bytes) {
  if (!model || model_bytes < kmm_model_bytes(precision, kern->d, n, tmax)) return false;
  if (m > 0 && (!ws || ws_bytes < kmm_query_bytes(precision, kern->d, n, m, tmax))) return false;
  p.precision = precision;
  p.kind = kern->kind;
  p.d = kern->d;
  p.square = false;
  p.n = n;
  p.m = m;
  p.npad = round_up(n, 32);
  p.mpad = round_up(m > 0 ? m : 1, 256);
  p.nchunks = p.npad / 32;
  p.ks = kmm_ksteps(precision, kern->d);
  p.tmax = tmax;
  p.ntb = (tmax + 15) / 16;
  p.sf = kern->outputscale;
  p.noise = kern->noise;
  char* c = (char*)model;
  p.xr = c;  c += align256((size_t)p.npad * p.ks * 64);
  p.nrm_b = (float*)c;  c += align256((size_t)p.npad * 4);
  carve_vfrag(p, c);
  c += kmm_vfrag_bytes(n, tmax);
  p.ctr = (double*)c;  c += align256((size_t)p.d * 8);
  p.cpart = (double*)c;  c += align256(colmean_scratch_doubles(n, p.d) * 8);
  if (m > 0) {
    char* w = (char*)ws;
    p.xc = w;  w += align256((size_t)p.mpad * p.ks * 64);
    p.nrm_a = (float*)w;  w += align256((size_t)p.mpad * 4);
    p.nrm64 = (double*)w;  w += align256((size_t)p.mpad * 8);
    p.part = (double*)w;
  } else {
    // preparing the model only: the FP64 norm scratch lives at the end of the model buffer
    p.xc = nullptr;
    p.nrm_a = nullptr;
    p.nrm64 = (double*)c;
    p.part = nullptr;
  }
  return true;
}

double profile_coordinate_scale(int kind) {
  return kind == GP_MATERN52 ? std::sqrt(5.0) * M_LOG2E : std::sqrt(0.5 * M_LOG2E);
}

static Scale make_scale(const gp_kernel* kern) {
  Scale s{};
  const double c = profile_coordinate_scale(kern->kind);
  for (int j = 0; j < kern->d; ++j) s.s[j] = c / kern->lengthscale[j];
  return s;
}

// set_centre: P is the b stream (the training points), whose column means become
// the centre of the mixed form's coordinates (p.ctr); otherwise P is query rows,
// prepared against the centre already in p.ctr.
static hipError_t prep_points(const KmmPlan& p, const Scale& sc, const double* P, int64_t rows,
                              int64_t rows_pad, void* xr, void* xc, float* nr, float* nc, bool set_centre,
                              hipStream_t st) {
  if (!p.nrm64 || !P || (!xr && !xc)) return hipErrorInvalidValue;
  const int mixed = p.precision == GP_PREC_BF16X3;
  if (mixed && (!p.ctr || (set_centre && !p.cpart))) return hipErrorInvalidValue;
  if (mixed && set_centre) {
    const hipError_t e = column_means(P, rows, p.d, p.cpart, p.ctr, st);
    if (e != hipSuccess) return e;
  }
  if (mixed) return launch_prep_points(P, p.ctr, rows, rows_pad, p.d, p.ks, sc, xr, xc, nullptr, st);
  const int thr = 256;
  prep_norm_fp32_kernel<<<(unsigned)((rows_pad + thr - 1) / thr), thr, 0, st>>>(P, rows, rows_pad, p.d, sc, p.nrm64);
  const int64_t nblk = rows_pad / 16;
  const int64_t total = nblk * p.ks * 64;
  prep_frag_fp32_kernel<<<(unsigned)((total + thr - 1) / thr), thr, 0, st>>>(P, p.nrm64, rows, nblk, p.d, p.ks, sc,
                                                                             (f32x4*)xr, (f32x4*)xc, nr, nc);
  return hipGetLastError();
}

hipError_t kmm_prepare(KmmPlan& p, const gp_kernel* kern, const double* X, const double* Z,
                       hipStream_t st) {
  if (p.precision == GP_PREC_FP64) return fp64_prepare(p, kern, X, Z, st);
  const Scale sc = make_scale(kern);
  if (p.square) {
    // one pass gives both sides; rows up to max(npad, mpad) so xc covers mpad
    const int64_t rows_pad = std::max(p.npad, p.mpad);
    return prep_points(p, sc, X, p.n, rows_pad, p.xr, p.xc, p.nrm_b, p.nrm_a, true, st);
  }
  hipError_t e = kmm_prepare_rows(p, kern, X, st);
  if (e != hipSuccess) return e;
  return kmm_prepare_cols(p, kern, Z, st);
}

hipError_t kmm_prepare_rows(KmmPlan& p, const gp_kernel* kern, const double* X, hipStream_t st) {
  if (p.precision == GP_PREC_FP64) return hipErrorInvalidValue;
  return prep_points(p, make_scale(kern), X, p.n, p.npad, p.xr, nullptr, p.nrm_b, nullptr, true, st);
}

hipError_t kmm_prepare_cols(KmmPlan& p, const gp_kernel* kern, const double* Z, hipStream_t st) {
  if (p.precision == GP_PREC_FP64) return hipErrorInvalidValue;
  return prep_points(p, make_scale(kern), Z, p.m, p.mpad, nullptr, p.xc, nullptr, p.nrm_a, false, st);
}

hipError_t prep_dist(const gp_kernel* kern, const double* X, int64_t n, int64_t rows_pad, int ks, const double* ctr,
                     void* xr, void* xc, double* nrm64, hipStream_t st) {
  if (!X || !ctr || !nrm64 || (!xr && !xc) || ks * 32 < 3 * kern->d + 6 || rows_pad % 64 != 0)
    return hipErrorInvalidValue;
  return launch_prep_points(X, ctr, n, rows_pad, kern->d, ks, make_scale(kern), xr, xc, nrm64, st);
}

template <int KS>
static void launch_one(bool mixed, int nt, int kind, int na, dim3 grid, const SweepArgs& a, hipStream_t st);

// BF16X3 K steps (32 wide) and FP32 K groups (16 wide) that are instantiated.
static bool dispatch_ks(int ks, int nt, int kind, bool mixed, int na, dim3 grid, const SweepArgs& a,
                        hipStream_t st) {
  if (mixed) {
    switch (ks) {
      case 2: launch_one<2>(true, nt, kind, na, grid, a, st); return true;
      case 4: launch_one<4>(true, nt, kind, na, grid, a, st); return true;
      case 5: launch_one<5>(true, nt, kind, na, grid, a, st); return true;
      case 7: launch_one<7>(true, nt, kind, na, grid, a, st); return true;
      case 13: launch_one<13>(true, nt, kind, na, grid, a, st); return true;
      default: return false;
    }
  }
  switch (ks) {
    case 1: launch_one<1>(false, nt, kind, na, grid, a, st); return true;
    case 2: launch_one<2>(false, nt, kind, na, grid, a, st); return true;
    case 3: launch_one<3>(false, nt, kind, na, grid, a, st); return true;
    case 4: launch_one<4>(false, nt, kind, na, grid, a, st); return true;
    case 8: launch_one<8>(false, nt, kind, na, grid, a, st); return true;
    default: return false;
  }
}

template <int KS, int NT, int KIND>
static void launch_form(bool mixed, int na, dim3 grid, const SweepArgs& a, hipStream_t st) {
  if constexpr (KS == 2 || KS == 4 || KS == 5 || KS == 7 || KS == 13) {
    if (mixed) {
      sweep_bf16x3_kernel<KS, NT, KIND><<<grid, 256, 0, st>>>(a);
      return;
    }
  }
  if constexpr (KS == 1 || KS == 2 || KS == 3 || KS == 4 || KS == 8) {
    if constexpr (pair_gain_f32(KS, NT, KIND) >= 0) {
      if (!mixed && na == 2) {
        sweep_fp32_kernel<KS, NT, KIND, 2><<<grid, 256, 0, st>>>(a);
        return;
      }
    }
    if (!mixed) sweep_fp32_kernel<KS, NT, KIND, 1><<<grid, 256, 0, st>>>(a);
  }
}

template <int KS>
static void launch_one(bool mixed, int nt, int kind, int na, dim3 grid, const SweepArgs& a, hipStream_t st) {
  const bool m52 = kind == GP_MATERN52;
  switch (nt) {
    case 1: m52 ? launch_form<KS, 1, GP_MATERN52>(mixed, na, grid, a, st)
                : launch_form<KS, 1, GP_RBF>(mixed, na, grid, a, st); break;
    case 2: m52 ? launch_form<KS, 2, GP_MATERN52>(mixed, na, grid, a, st)
                : launch_form<KS, 2, GP_RBF>(mixed, na, grid, a, st); break;
    case 3: m52 ? launch_form<KS, 3, GP_MATERN52>(mixed, na, grid, a, st)
                : launch_form<KS, 3, GP_RBF>(mixed, na, grid, a, st); break;
    default: m52 ? launch_form<KS, 4, GP_MATERN52>(mixed, na, grid, a, st)
                : launch_form<KS, 4, GP_RBF>(mixed, na, grid, a, st); break;
  }
}

// The mixed form's V operand for one launch, and its workgroups.
static VSet v_set(const KmmPlan& p, const double* V, int64_t ldv, int t, bool row_independent, const double* col0,
                  int64_t* blocks) {
  const SplitChoice sc = choose_split(p.npad, p.mpad, (t + 15) / 16, row_independent, p.ks, true);
  const int ntb = sc.groups * sc.nt;  // vf holds whole launch groups (zero padded)
  // one chunk per wave until the chip is full (four waves per SIMD), then up to eight
  const int per = (int)std::max<int64_t>(1, std::min<int64_t>(8, p.nchunks * ntb / 4096));
  *blocks = ((p.nchunks + per - 1) / per * ntb * 64 + 255) / 256;
  return VSet{V, ldv, col0, p.vpart, p.vinv, p.n, p.nchunks, t, ntb, per, (bf16x8*)p.vf};
}

hipError_t kmm_prepare_v(const KmmPlan& p, const double* V, int64_t ldv, int t, bool row_independent,
                         hipStream_t st, const double* col0) {
  if (t < 1 || t > p.tmax || !p.vf || !V) return hipErrorInvalidValue;
  if (p.precision == GP_PREC_BF16X3) {
    if (!p.vinv || !p.vpart) return hipErrorInvalidValue;
    int64_t blocks;
    const VSet vs = v_set(p, V, ldv, t, row_independent, col0, &blocks);
    vmax_partial_kernel<<<dim3(kVParts, (unsigned)t), 256, 0, st>>>(V, ldv, col0, p.n, p.vpart);
    prep_v_f16x3_kernel<<<(unsigned)blocks, 256, 0, st>>>(vs);
  } else {
    const int ntb = (t + 15) / 16;
    const SplitChoice sc = choose_split(p.npad, p.mpad, ntb, row_independent, p.ks, false);
    const int ntb_alloc = sc.groups * sc.nt, thr = 256;
    const int64_t total = p.nchunks * ntb_alloc * 2 * 64;
    prep_v_fp32_kernel<<<(unsigned)((total + thr - 1) / thr), thr, 0, st>>>(V, ldv, col0, p.n, t, p.nchunks,
                                                                             ntb_alloc, (f32x4*)p.vf);
  }
  return hipGetLastError();
}

template <int KS, int FULL, int REST>
static void launch_wide_form(int kind, dim3 grid, const WideArgs& a, hipStream_t st) {
  if (kind == GP_MATERN52)
    wide_cross_bf16x3_kernel<KS, FULL, REST, GP_MATERN52><<<grid, 256, 0, st>>>(a);
  else
    wide_cross_bf16x3_kernel<KS, FULL, REST, GP_RBF><<<grid, 256, 0, st>>>(a);
}

template <int KS>
static void launch_wide(int kind, dim3 grid, const WideArgs& a, hipStream_t st) {
  // 4 FULL + REST >= ntb column blocks; up to three of a form's are beyond the last
  const int ntb = a.ntb;
  if (ntb == 1) return launch_wide_form<KS, 0, 1>(kind, grid, a, st);
  if (ntb <= 3) return launch_wide_form<KS, 0, 3>(kind, grid, a, st);
  if (ntb <= 5) return launch_wide_form<KS, 1, 1>(kind, grid, a, st);
  if (ntb <= 9) return launch_wide_form<KS, 2, 1>(kind, grid, a, st);
  if (ntb <= 13) return launch_wide_form<KS, 3, 1>(kind, grid, a, st);
  if (ntb <= 17) return launch_wide_form<KS, 4, 1>(kind, grid, a, st);
  launch_wide_form<KS, 5, 0>(kind, grid, a, st);
}

// Row-independent BF16X3 cross products (prediction): the wide sweep, same splits and partials.
static hipError_t kmm_sweep_wide(const KmmPlan& p, int t, const SplitChoice& sc, double* out, int64_t ldo,
                                 hipStream_t st) {
  WideArgs a;
  a.xr = p.xr;
  a.xc = p.xc;
  a.vf = p.vf;
  a.part = p.part;
  a.mpad = p.mpad;
  a.nchunks = p.nchunks;
  a.cps = sc.cps;
  a.nsplit = sc.nsplit;
  a.t = t;
  a.m = p.m;
  a.ntb = (t + 15) / 16;
  a.vstride = sc.groups * sc.nt;  // the V fragments hold whole launch groups
  a.tpad = a.ntb * 16;
  a.rgroups = (int)std::max<int64_t>(1, (p.m + 63) / 64);  // live 64-row groups (mpad is a multiple of 256)
  a.f32part = sc.cps <= kFlush ? 1 : 0;
  const dim3 grid((unsigned)(a.rgroups * ((sc.nsplit + 7) / 8 * 8)));
  SweepTiming::Rec rec{};
  bool timed = false;
  {
    std::lock_guard<std::mutex> g(timing().mu);
    timed = timing().on && !p.no_timing;
  }
  if (timed) {
    hipError_t e = hipEventCreate(&rec.a);
    if (e == hipSuccess) e = hipEventCreate(&rec.b);
    if (e == hipSuccess) e = hipEventRecord(rec.a, st);
    if (e != hipSuccess) return e;
  }
  switch (p.ks) {
    case 2: launch_wide<2>(p.kind, grid, a, st); break;
    case 4: launch_wide<4>(p.kind, grid, a, st); break;
    case 5: launch_wide<5>(p.kind, grid, a, st); break;
    case 7: launch_wide<7>(p.kind, grid, a, st); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (timed) {
    e = hipEventRecord(rec.b, st);
    if (e != hipSuccess) return e;
    rec.flops = 2.0 * (double)p.m * (double)p.n * (double)(p.d + t);
    rec.n = p.n;
    rec.m = p.m;
    rec.t = t;
    std::lock_guard<std::mutex> g(timing().mu);
    timing().recs.push_back(rec);
  }
  const dim3 egrid((unsigned)((p.m + 63) / 64), (unsigned)t);
  if (a.f32part)
    wide_epilogue_kernel<float><<<egrid, 256, 0, st>>>((const float*)p.part, sc.nsplit, a.tpad, p.mpad, p.m, p.sf,
                                                       p.vinv, out, ldo);
  else
    wide_epilogue_kernel<double><<<egrid, 256, 0, st>>>(p.part, sc.nsplit, a.tpad, p.mpad, p.m, p.sf, p.vinv, out,
                                                        ldo);
  return hipGetLastError();
}

hipError_t kmm_sweep(const KmmPlan& p, int t, const double* Vdiag, int64_t ldv, double* out, int64_t ldo,
                     hipStream_t st, bool row_independent, const DotPartials& dot) {
  if (t < 1 || t > p.tmax || (dot.part && !p.square)) return hipErrorInvalidValue;
  if (!p.xr || !p.xc || !p.nrm_b || !p.nrm_a || !p.vf || !p.part || !out) return hipErrorInvalidValue;
  const bool mixed = p.precision == GP_PREC_BF16X3;
  const int ntb = (t + 15) / 16;
  const SplitChoice sc = choose_split(p.npad, p.mpad, ntb, row_independent, p.ks, p.precision == GP_PREC_BF16X3);
  if (row_independent && mixed && !p.square && ntb <= kWideBlocks && p.ks <= 7)
    return kmm_sweep_wide(p, t, sc, out, ldo, st);
  SweepArgs a;
  a.xr = p.xr;
  a.xc = p.xc;
  a.nrm_b = p.nrm_b;
  a.nrm_a = p.nrm_a;
  a.vf = p.vf;
  a.part = p.part;
  a.mpad = p.mpad;
  a.nchunks = p.nchunks;
  a.cps = sc.cps;
  a.ntb = sc.groups * sc.nt;
  a.tpad = sc.tpad;
  a.t = t;
  a.f32part = sc.cps <= kFlush ? 1 : 0;
  a.square = p.square ? 1 : 0;
  const int na = mixed ? na_of(p.ks, sc.nt) : na_f32(p.ks, sc.nt, p.kind, p.mpad, sc.nsplit, sc.groups);
  dim3 grid((unsigned)(p.mpad / (64 * na)), (unsigned)sc.nsplit, (unsigned)sc.groups);
  SweepTiming::Rec rec{};
  bool timed = false;
  {
    std::lock_guard<std::mutex> g(timing().mu);
    timed = timing().on && !p.no_timing;
  }
  if (timed) {
    hipError_t e = hipEventCreate(&rec.a);
    if (e == hipSuccess) e = hipEventCreate(&rec.b);
    if (e == hipSuccess) e = hipEventRecord(rec.a, st);
    if (e != hipSuccess) return e;
  }
  if (!dispatch_ks(p.ks, sc.nt, p.kind, mixed, na, grid, a, st)) return hipErrorInvalidValue;
  if (timed) {
    hipError_t e = hipEventRecord(rec.b, st);
    if (e != hipSuccess) return e;
    rec.flops = 2.0 * (double)p.m * (double)p.n * (double)(p.d + t);
    rec.n = p.n;
    rec.m = p.m;
    rec.t = t;
    std::lock_guard<std::mutex> g(timing().mu);
    timing().recs.push_back(rec);
  }
  const dim3 egrid((unsigned)((p.m + dot.rows - 1) / dot.rows), (unsigned)t);
  const double diag = p.square ? p.sf + p.noise : 0.0;
  const double* const inv = mixed ? p.vinv : nullptr;
  const double* const Vd = p.square ? Vdiag : nullptr;
  if (a.f32part)
    kmm_epilogue_kernel<float><<<egrid, 256, 0, st>>>((const float*)p.part, sc.nsplit, sc.tpad, p.mpad, p.m, t, p.sf,
                                                      diag, inv, Vd, ldv, out, ldo, dot.rows, dot.part);
  else
    kmm_epilogue_kernel<double><<<egrid, 256, 0, st>>>(p.part, sc.nsplit, sc.tpad, p.mpad, p.m, t, p.sf, diag, inv, Vd,
                                                       ldv, out, ldo, dot.rows, dot.part);
  return hipGetLastError();
}

hipError_t kmm_product(KmmPlan& p, const gp_kernel* kern, const double* X, const double* Z, const double* V,
                       int64_t ldv, int t, double* out, int64_t ldo, hipStream_t st) {
  const bool row_independent = !p.square;
  if (p.precision != GP_PREC_BF16X3) {
    const hipError_t e = kmm_prepare(p, kern, X, Z, st);
    return e != hipSuccess ? e : kmm_apply(p, V, ldv, t, out, ldo, st, row_independent);
  }
  if (t < 1 || t > p.tmax || !p.vf || !V || !X || (!p.square && !Z) || !p.ctr || !p.cpart || !p.vinv || !p.vpart ||
      !p.xr || !p.xc)
    return hipErrorInvalidValue;
  const Scale sc = make_scale(kern);
  const int64_t nblk = colmean_blocks(p.n), rpb = (p.n + nblk - 1) / nblk;
  prep_reduce_f16x3_kernel<<<(unsigned)(nblk + (int64_t)kVParts * t), 256, 0, st>>>(X, p.n, p.d, rpb, (int)nblk,
                                                                                   p.cpart, V, ldv, p.vpart);
  Centre ce{p.ctr, p.cpart, (int)nblk, p.n};
  if (nblk > kMeanFold) {
    colmean_final_kernel<<<(unsigned)((p.d + kMeanCols - 1) / kMeanCols), 256, 0, st>>>(p.cpart, (int)nblk, p.d, p.n,
                                                                                      p.ctr);
    ce.part = nullptr;
  }
  // the square case prepares both sides at once; rows up to max(npad, mpad) so xc covers mpad
  const int64_t xrows = p.square ? std::max(p.npad, p.mpad) : p.npad, zrows = p.square ? 0 : p.mpad;
  if (xrows % kPrepPts != 0 || zrows % kPrepPts != 0) return hipErrorInvalidValue;
  const PointSet px{X, p.n, (bf16x8*)p.xr, p.square ? (bf16x8*)p.xc : nullptr, nullptr};
  const PointSet pz{Z, p.m, nullptr, (bf16x8*)p.xc, nullptr};
  int64_t vblocks;
  const VSet vs = v_set(p, V, ldv, t, row_independent, nullptr, &vblocks);
  const int64_t nbx = xrows / kPrepPts, nbz = zrows / kPrepPts;
  const unsigned grid = (unsigned)(nbx + nbz + vblocks);
  const size_t lds = prep_points_lds(p.ks);
#define GPK_PREP(NS) prep_operands_f16x3_kernel<NS><<<grid, 256, lds, st>>>(px, pz, nbx, nbz, ce, p.d, p.ks, sc, vs)
  switch ((p.d + 15) / 16) {
    case 1: GPK_PREP(1); break;
    case 2: GPK_PREP(2); break;
    case 3: GPK_PREP(3); break;
    case 4: GPK_PREP(4); break;
    default: GPK_PREP(8); break;
  }
#undef GPK_PREP
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : kmm_sweep(p, t, V, ldv, out, ldo, st, row_independent);
}

hipError_t kmm_apply(const KmmPlan& p, const double* V, int64_t ldv, int t, double* out, int64_t ldo,
                     hipStream_t st, bool row_independent, const DotPartials& dot) {
  if (p.precision == GP_PREC_FP64) return dot.part ? hipErrorInvalidValue : fp64_sweep(p, V, ldv, t, out, ldo, st);
  hipError_t e = kmm_prepare_v(p, V, ldv, t, row_independent, st);
  if (e != hipSuccess) return e;
  return kmm_sweep(p, t, V, ldv, out, ldo, st, row_independent, dot);
}

}  // namespace gpk
