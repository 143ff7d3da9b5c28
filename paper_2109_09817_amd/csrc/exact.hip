// Exact GP on a subset (the AltBBMM hyperparameter protocol, Sec. 3.2 and
// Sec. 4: the hyperparameters come from a full GP on a random subset of the
// training molecules).  Dense FP64 throughout:
//
//   K_hat = L L^T (blocked right-looking Cholesky, 64-wide panels)
//   X = L^{-1}                   (by doubling the inverted diagonal blocks)
//   K_hat^{-1} = X^T X           (lower tiles)
//   omega = K_hat^{-1} y
//   L(theta) = -1/2 y^T omega - sum_a log L_aa - n/2 log 2 pi       (Eq. 2)
//   dL/dlog theta = 1/2 sum_ab (omega omega^T - K_hat^{-1})_ab dK_hat_ab/dlog theta
//
// with dK/dlog l_j = psi(r) (dx_j / l_j)^2, psi(r) = (5/3) s_f (1 + sqrt5 r)
// e^{-sqrt5 r} (Matern-5/2; RBF: k), dK/dlog s_f = K and dK_hat/dlog sigma^2
// = sigma^2 I.  Every O(n^3) step is a sequence of FP64 tile products on the
// matrix cores, the operands staged in LDS: the panels of the Cholesky
// factorisation in 64 x 64 tiles (k = 64 inside a super-panel of 256 columns, 256
// for the next one), its trailing updates in 128 x 128 tiles beside the next
// diagonal blocks, the inverse and the large-rank products in 128 x 128 tiles where
// these fill the chip and 64 x 64 below.  Triangular solves against a 64 x 64
// diagonal block multiply by its inverse (formed in LDS by one workgroup), so
// that they are tile products too.
#include <algorithm>
#include <cmath>
#include <vector>

#include "api_common.h"
#include "solver.h"

namespace gpk {

constexpr int kEb = 64;         // panel width and tile edge
constexpr int kExactMaxD = 64;  // features (the derivative sweep keeps a row of d in LDS)
constexpr int64_t kExactMaxN = 65536;

// ---------------------------------------------------------------- K_hat

// A[a n + b] = s_f m(r_ab) + sigma^2 [a == b] by direct differences.  sc[f]:
// Matern sqrt5 / l_f (so u = sqrt5 r), RBF 1 / l_f.
template <int KIND>
__global__ __launch_bounds__(256) void form_khat_kernel(const double* __restrict__ X, int64_t n, int d,
                                                        const double* __restrict__ sc, double sf, double noise,
                                                        double* __restrict__ A) {
  __shared__ double xa[kEb][33];
  __shared__ double xbT[32][kEb];
  const int64_t a0 = (int64_t)blockIdx.y * kEb, b0 = (int64_t)blockIdx.x * kEb;
  const int c = threadIdx.x % kEb, rb = threadIdx.x / kEb;
  double acc[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) acc[j] = 0.0;
  for (int f0 = 0; f0 < d; f0 += 32) {
    __syncthreads();
    for (int e = threadIdx.x; e < kEb * 32; e += 256) {
      const int row = e / 32, f = e % 32;
      const bool fin = f0 + f < d;
      xa[row][f] = (a0 + row < n && fin) ? X[(a0 + row) * d + f0 + f] * sc[f0 + f] : 0.0;
      xbT[f][row] = (b0 + row < n && fin) ? X[(b0 + row) * d + f0 + f] * sc[f0 + f] : 0.0;
    }
    __syncthreads();
    for (int f = 0; f < 32; ++f) {
      const double xb = xbT[f][c];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const double t = xa[rb + 4 * j][f] - xb;
        acc[j] = fma(t, t, acc[j]);
      }
    }
  }
  const int64_t b = b0 + c;
  if (b >= n) return;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int64_t a = a0 + rb + 4 * j;
    if (a >= n) continue;
    double m;
    if constexpr (KIND == GP_MATERN52) {
      const double u = sqrt(acc[j]);
      m = (1.0 + u + u * u / 3.0) * exp(-u);
    } else {
      m = exp(-0.5 * acc[j]);
    }
    A[a * n + b] = sf * m + (a == b ? noise : 0.0);
  }
}

// ---------------------------------------------------------------- Cholesky

typedef double f64x4 __attribute__((ext_vector_type(4)));

// v of lane `lane` (a constant), as a wave-uniform value.
__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

constexpr int kDb = 16;         // sub-block edge of the diagonal factorisation
constexpr int kDbLd = kEb + 2;  // LDS pitch: the MFMA's 16-row operand reads hit distinct banks

// Cholesky of a 16 x 16 block and the inverse of its factor, by one wave in
// registers: lane l holds row l % 16 in a (lower part; the upper part is
// ignored on entry and zero on return) and column l % 16 of the inverse in x.
// Entries of other lanes are read as scalars.  base: global index of row 0.
__device__ __forceinline__ void chol_inverse_16(double (&a)[kDb], double (&x)[kDb], int lr, int base, int& bad) {
#pragma unroll
  for (int k = 0; k < kDb; ++k) {
    double p = lane_value(a[k], k);
    if (!(p > 0.0) || !isfinite(p)) {
      if (bad == 0) bad = base + k + 1;
      p = 1.0;
    }
    const double piv = sqrt(p);
    const double l = a[k] / piv;
    a[k] = lr == k ? piv : (lr > k ? l : 0.0);
#pragma unroll
    for (int c = k + 1; c < kDb; ++c) a[c] = fma(-a[k], lane_value(a[k], c), a[c]);
  }
#pragma unroll
  for (int r = 0; r < kDb; ++r) x[r] = r == lr ? 1.0 : 0.0;
#pragma unroll
  for (int r = 0; r < kDb; ++r) {
    x[r] /= lane_value(a[r], r);
#pragma unroll
    for (int q = r + 1; q < kDb; ++q) x[q] = fma(-lane_value(a[r], q), x[r], x[q]);
  }
}

// Cholesky of the diagonal block A[j0.., j0..] (jb <= 64 rows) in LDS, the
// block outside jb padded with the identity; writes L (lower, zero above the
// diagonal) and L^{-1} (64 x 64 row-major, into Dinv).  A pivot that is not
// positive records its global index + 1 in *info (the first one only)
// and continues with 1, so that every later step stays finite and bounded.
//
// One workgroup on the factorisation's critical path: the time is the length
// of its serial chain.  Four 16-column steps: wave 0 factors and inverts the
// 16 x 16 diagonal block in registers, the waves multiply the rows below by
// that inverse and update the trailing 16 x 16 tiles on the FP64 matrix cores
// (lane l supplies P(l % 16, l / 16) and Q(l / 16, l % 16), and receives rows
// l / 16 + 4 i); 3 barriers a step.  The inverse's blocks below the diagonal
// follow block diagonal by block diagonal, X_ij = -X_ii sum_k L_ik X_kj.
// Column by column over all 64 (128 barriers, then 64 dependent rows of the
// inverse) it took 74 us; this form: 29 us in a launch of its own (n = 7,503: 118 of
// them, 30.1 -> 24.8 ms), 31 to 35 us in the fused launch below.
__device__ __forceinline__ void potrf_diag(double* __restrict__ A, int64_t n, int64_t j0, int jb, int* __restrict__ info,
                                           double* __restrict__ Dinv, double* Ls, double* Xs) {
  constexpr int kPer = kEb * kEb / 256;
  const int tid = threadIdx.x;
  {
    double v[kPer];  // every load in flight before the first LDS write
#pragma unroll
    for (int it = 0; it < kPer; ++it) {
      const int e = tid + 256 * it, r = e / kEb, c = e % kEb;
      v[it] = (r < jb && c < jb) ? A[(j0 + r) * n + j0 + c] : (r == c ? 1.0 : 0.0);
    }
#pragma unroll
    for (int it = 0; it < kPer; ++it) {
      const int e = tid + 256 * it;
      Ls[e / kEb * kDbLd + e % kEb] = v[it];
      Xs[e / kEb * kDbLd + e % kEb] = 0.0;
    }
  }
  const int lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  constexpr int kNb = kEb / kDb;
  int bad = 0;  // wave 0 only
  __syncthreads();
  for (int b = 0; b < kNb; ++b) {
    const int c0 = kDb * b;
    if (wave == 0) {
      double a[kDb], x[kDb];
#pragma unroll
      for (int j = 0; j < kDb; ++j) a[j] = Ls[(c0 + lr) * kDbLd + c0 + j];
      chol_inverse_16(a, x, lr, (int)j0 + c0, bad);
      if (lk == 0) {
#pragma unroll
        for (int j = 0; j < kDb; ++j) {
          Ls[(c0 + lr) * kDbLd + c0 + j] = a[j];
          Xs[(c0 + j) * kDbLd + c0 + lr] = x[j];
        }
      }
    }
    __syncthreads();
    const int below = kNb - 1 - b;
    if (wave < below) {  // row block b + 1 + wave: L = A X_bb^T
      const int r0 = c0 + kDb * (1 + wave);
      f64x4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 4; ++s)
        d = __builtin_amdgcn_mfma_f64_16x16x4f64(Ls[(r0 + lr) * kDbLd + c0 + 4 * s + lk],
                                                 Xs[(c0 + lr) * kDbLd + c0 + 4 * s + lk], d, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) Ls[(r0 + lk + 4 * i) * kDbLd + c0 + lr] = d[i];
    }
    __syncthreads();
    for (int q = wave; q < below * (below + 1) / 2; q += 4) {  // trailing tiles (ri, cj), cj <= ri
      const int ri = q >= 3 ? 2 : (q >= 1 ? 1 : 0), cj = q - ri * (ri + 1) / 2;
      const int r0 = c0 + kDb * (1 + ri), q0 = c0 + kDb * (1 + cj);
      f64x4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 4; ++s)
        d = __builtin_amdgcn_mfma_f64_16x16x4f64(Ls[(r0 + lr) * kDbLd + c0 + 4 * s + lk],
                                                 Ls[(q0 + lr) * kDbLd + c0 + 4 * s + lk], d, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) Ls[(r0 + lk + 4 * i) * kDbLd + q0 + lr] -= d[i];
    }
    __syncthreads();
  }
  for (int e = tid; e < kEb * kEb; e += 256) {
    const int r = e / kEb, c = e % kEb;
    if (r < jb && c < jb) A[(j0 + r) * n + j0 + c] = c <= r ? Ls[r * kDbLd + c] : 0.0;
  }
  if (tid == 0 && bad != 0 && *info == 0) *info = bad;
  for (int dist = 1; dist < kNb; ++dist) {
    if (wave < kNb - dist) {
      const int j = wave, i = wave + dist;
      f64x4 t = {0.0, 0.0, 0.0, 0.0};
      for (int k = j; k < i; ++k)
#pragma unroll
        for (int s = 0; s < 4; ++s)
          t = __builtin_amdgcn_mfma_f64_16x16x4f64(Ls[(kDb * i + lr) * kDbLd + kDb * k + 4 * s + lk],
                                                   Xs[(kDb * k + 4 * s + lk) * kDbLd + kDb * j + lr], t, 0, 0, 0);
      f64x4 d = {0.0, 0.0, 0.0, 0.0};  // register s of t holds its rows 4 s + l / 16
#pragma unroll
      for (int s = 0; s < 4; ++s)
        d = __builtin_amdgcn_mfma_f64_16x16x4f64(Xs[(kDb * i + lr) * kDbLd + kDb * i + 4 * s + lk], t[s], d, 0, 0, 0);
#pragma unroll
      for (int s = 0; s < 4; ++s) Xs[(kDb * i + lk + 4 * s) * kDbLd + kDb * j + lr] = -d[s];
    }
    __syncthreads();
  }
  for (int e = tid; e < kEb * kEb; e += 256) Dinv[e] = Xs[e / kEb * kDbLd + e % kEb];
}

// ---------------------------------------------------------------- tile updates

// C[R + r][Cc + c] -= sum_{k < kb} P(r, k) Q(c, k) (ASSIGN: =) over a set of
// 64 x 64 tiles (k in chunks of 64 staged in LDS in turn), with
//   P(r, k) = Pm[(R + r) ldp + p0 + k],  Q(c, k) = Qm[(qc + c) ldq + q0 + k]
// where qc = Cc (qfix < 0) or qfix.  Tile (ti, tj) has R = rbase + 64 ti, Cc =
// cbase + 64 tj; LOWER enumerates tj <= ti of the nrt x nct (nct <= nrt)
// rectangle, otherwise all of it.  Output rows and columns at or beyond
// n are skipped (their operands read as 0).  Every operand is read before
// the tile is written, so C's tile may be one of the operand tiles (never
// another workgroup's).  The products run on the FP64 matrix cores
// (v_mfma_f64_16x16x4: lane l supplies P(row l % 16, k l / 16) and Q(k l / 16,
// column l % 16) and receives rows l / 16 + 4 i of column l % 16); wave w
// owns the 32 x 32 quadrant (w / 2, w % 2).  Operands in LDS keep the
// orientation of their source rows, so that a wave's staging writes are
// contiguous: k-major [k][x] (pitch 80 doubles) when the source runs along x,
// x-major [x][k] (pitch 66) when it runs along k, as both operands do here.  Both
// pitches put the 32 lanes of a half-wave on distinct banks for the operand reads.
constexpr int kKMajorLd = kEb + 16;
constexpr int kXMajorLd = kEb + 2;

template <bool KMAJOR>
__device__ __forceinline__ int lds_at(int k, int x) {
  return KMAJOR ? k * kKMajorLd + x : x * kXMajorLd + k;
}

// Tile b of a lower triangle counted row by row: (0, 0), (1, 0), (1, 1), ...
__device__ __forceinline__ void lower_tile(int64_t b, int64_t& ti, int64_t& tj) {
  ti = (int64_t)((sqrt(8.0 * (double)b + 1.0) - 1.0) * 0.5);
  while ((ti + 1) * (ti + 2) / 2 <= b) ++ti;
  while (ti * (ti + 1) / 2 > b) --ti;
  tj = b - ti * (ti + 1) / 2;
}

template <bool LOWER, bool ASSIGN>
__global__ __launch_bounds__(256) void tile_update_kernel(const double* Pm, int64_t ldp, int64_t p0, const double* Qm,
                                                          int64_t ldq, int64_t qfix, int64_t q0, double* Cm, int64_t n,
                                                          int kb, int64_t rbase, int64_t cbase, int nrt, int nct) {
  __shared__ double Ps[kEb * kXMajorLd], Qs[kEb * kXMajorLd];  // P(r, k) and Q(c, k) at lds_at<false>(k, r or c)
  int64_t ti, tj;
  // Workgroup h runs on XCD h % 8; each XCD takes a contiguous run of tiles
  // (consecutive tiles of a tile row share their P panel in that XCD's L2).
  const int64_t tri = LOWER ? (int64_t)nct * (nct + 1) / 2 : 0;  // the nct x nct part
  const int64_t T = LOWER ? tri + (int64_t)(nrt - nct) * nct : (int64_t)nrt * nct;
  const int64_t h = blockIdx.x, xcd = h & 7, q8 = T >> 3, rem8 = T & 7;
  const int64_t b = xcd * q8 + (xcd < rem8 ? xcd : rem8) + (h >> 3);
  if (LOWER && b < tri) {
    lower_tile(b, ti, tj);
  } else {
    ti = (b - tri) / nct;
    tj = b - tri - ti * nct;
    if (LOWER) ti += nct;
  }
  const int64_t R = rbase + kEb * ti, Cc = cbase + kEb * tj;
  const int64_t qc = qfix < 0 ? Cc : qfix;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = 32 * (wave >> 1), c0 = 32 * (wave & 1);
  const int lr = lane & 15, lk = lane >> 4;
  f64x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  // Each thread stages 16 elements of each operand per 64-wide k chunk; the
  // loads of chunk c + 1 are in flight while chunk c is multiplied.
  constexpr int kPer = kEb * kEb / 256;
  double pv[kPer], qv[kPer];
  auto load = [&](int kc) {
#pragma unroll
    for (int it = 0; it < kPer; ++it) {
      const int e = (int)threadIdx.x + 256 * it;
      const int x = e / kEb, k = e % kEb;  // consecutive threads: consecutive k
      pv[it] = kc + k < kb && R + x < n ? Pm[(R + x) * ldp + p0 + kc + k] : 0.0;
      qv[it] = kc + k < kb && Cc + x < n ? Qm[(qc + x) * ldq + q0 + kc + k] : 0.0;
    }
  };
  auto store = [&]() {
#pragma unroll
    for (int it = 0; it < kPer; ++it) {
      const int e = (int)threadIdx.x + 256 * it;
      Ps[lds_at<false>(e % kEb, e / kEb)] = pv[it];
      Qs[lds_at<false>(e % kEb, e / kEb)] = qv[it];
    }
  };
  load(0);
  for (int kc = 0; kc < kb; kc += kEb) {
    if (kc > 0) __syncthreads();  // every wave is done with the previous chunk
    store();
    __syncthreads();
    if (kc + kEb < kb) load(kc + kEb);
#pragma unroll 4
    for (int k = 0; k < kEb; k += 4) {
      const double a0 = Ps[lds_at<false>(k + lk, r0 + lr)], a1 = Ps[lds_at<false>(k + lk, r0 + 16 + lr)];
      const double q0v = Qs[lds_at<false>(k + lk, c0 + lr)], q1v = Qs[lds_at<false>(k + lk, c0 + 16 + lr)];
      acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, q0v, acc[0][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, q1v, acc[0][1], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, q0v, acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, q1v, acc[1][1], 0, 0, 0);
    }
  }
  // the subtracting form reads all 16 of its C entries before writing any
  double old[2][2][4];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t row = R + r0 + 16 * rb + lk + 4 * i, col = Cc + c0 + 16 * cb + lr;
        old[rb][cb][i] = (!ASSIGN && row < n && col < n) ? Cm[row * n + col] : 0.0;
      }
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t row = R + r0 + 16 * rb + lk + 4 * i, col = Cc + c0 + 16 * cb + lr;
        if (row < n && col < n) Cm[row * n + col] = ASSIGN ? acc[rb][cb][i] : old[rb][cb][i] - acc[rb][cb][i];
      }
}

template <bool LOWER, bool ASSIGN>
static hipError_t tile_update(const double* Pm, int64_t ldp, int64_t p0, const double* Qm, int64_t ldq, int64_t qfix,
                              int64_t q0, double* Cm, int64_t n, int kb, int64_t rbase, int64_t cbase, int nrt, int nct,
                              hipStream_t st) {
  const int64_t tiles =
      LOWER ? (int64_t)nct * (nct + 1) / 2 + (int64_t)(nrt - nct) * nct : (int64_t)nrt * nct;
  if (tiles <= 0) return hipSuccess;
  tile_update_kernel<LOWER, ASSIGN><<<(unsigned)tiles, 256, 0, st>>>(Pm, ldp, p0, Qm, ldq, qfix, q0, Cm, n, kb, rbase,
                                                                     cbase, nrt, nct);
  return hipGetLastError();
}

// General FP64 products on the matrix cores.  C (m x nn, row-major with ldc)
// = A B or = -A B (-= A B only where potrf_update_kernel stores a tile):
//   A(i, k) = TA ? A[k lda + i] : A[i lda + k], B(k, j) = TB ? B[j ldb + k] : B[k ldb + j].
// LOWER computes only the tiles with tj <= ti (m = nn).  Rows and columns
// beyond the matrices read as zero or as some valid row; nothing outside C's
// m x nn block is written.  tri skips the k range where an operand is zero:
//   kTriA: A is lower triangular, row tile R takes k < R + edge;
//   kTriAt: A is the transpose of a lower triangle, row tile R takes k >= R;
//   kTriB: B is lower triangular, column tile Cc takes k >= Cc
// (each operand zero above the diagonal inside its diagonal tiles).
// Batches (blockIdx.y = p) shift the three matrices by p times their strides;
// with mstep > 0 the batch's rows end at m - p mstep (the ragged last block of
// a block-diagonal sweep), and under kTriA so does its k.
enum Tri { kTriNone = 0, kTriA, kTriAt, kTriB };
enum GemmMode { kAssign = 0, kSubtract, kNegate };

// The order of k puts the large entries near a triangle's diagonal last, so
// that the many small ones are summed before they meet a large partial sum: in
// X^T X, taken from the diagonal outwards, positive terms below half a unit of
// the running sum were lost one by one (the log s_f derivative, a trace, was
// off by 2e-13 at n = 7,503 instead of 4e-16).
__device__ __forceinline__ bool gemm_descends(int tri) { return tri == kTriAt || tri == kTriB; }

struct GemmArgs {
  const double* A;
  int64_t lda, sA;
  const double* B;
  int64_t ldb, sB;
  double* C;
  int64_t ldc, sC;
  int64_t m, nn, kk;
  int64_t mmax, mstep;  // batches: rows of batch p = min(mmax, m - p mstep)
  int nrt, nct, tri;
};

// Tile (ti, tj) and k range of this workgroup; false when it has no rows.
// Workgroup h runs on XCD h % 8.  Each XCD takes a contiguous run of the tile
// order, so that its tiles share panels in its L2: rectangles go through
// groups of 8 tile columns, row by row (under kTriA the long rows first); under
// kTriB, whose columns differ in length, through groups of 8 tile rows, so that
// every XCD gets all lengths.  Lower triangles run along tile rows; under
// kTriAt, whose rows differ in length, they are dealt out round-robin.
template <bool LOWER, int EDGE>
__device__ __forceinline__ bool gemm_tile(const GemmArgs& g, int64_t m, int64_t kk_all, int64_t& R, int64_t& Cc,
                                          int64_t& k0, int64_t& kn) {
  const int64_t T = LOWER ? (int64_t)g.nrt * (g.nrt + 1) / 2 : (int64_t)g.nrt * g.nct;
  const int64_t h = blockIdx.x, xcd = h & 7, q8 = T >> 3, rem8 = T & 7;
  const int64_t b = LOWER && g.tri == kTriAt ? h : xcd * q8 + (xcd < rem8 ? xcd : rem8) + (h >> 3);
  int64_t ti, tj;
  if (LOWER) {
    lower_tile(b, ti, tj);
  } else if (g.tri == kTriB) {
    const int64_t grp = b / (8 * (int64_t)g.nct), rest = b - grp * 8 * g.nct;
    const int64_t width = g.nrt - 8 * grp < 8 ? g.nrt - 8 * grp : 8;
    tj = rest / width;
    ti = 8 * grp + rest - tj * width;
  } else {
    const int64_t grp = b / (8 * (int64_t)g.nrt), rest = b - grp * 8 * g.nrt;
    const int64_t width = g.nct - 8 * grp < 8 ? g.nct - 8 * grp : 8;
    ti = rest / width;
    tj = 8 * grp + rest - ti * width;
    if (g.tri == kTriA) ti = g.nrt - 1 - ti;
  }
  R = EDGE * ti;
  Cc = EDGE * tj;
  k0 = g.tri == kTriAt ? R : (g.tri == kTriB ? Cc : 0);
  kn = g.tri == kTriA && R + EDGE < kk_all ? R + EDGE : kk_all;
  return R < m;
}

// 64 x 64 output tiles, k in chunks of 64 staged in LDS as in the tile kernel above.
template <bool TA, bool TB, bool LOWER, int MODE>
__global__ __launch_bounds__(256) void gemm64_f64_kernel(GemmArgs g) {
  static_assert(MODE != kSubtract, "the tile is stored, not added to");
  __shared__ double As[kEb * kKMajorLd];  // A(r, k) at lds_at<TA>(k, r)
  __shared__ double Bs[kEb * kKMajorLd];  // B(k, c) at lds_at<!TB>(k, c)
  const int64_t p = blockIdx.y;
  const double* A = g.A + p * g.sA;
  const double* B = g.B + p * g.sB;
  double* C = g.C + p * g.sC;
  const int64_t m = g.mstep > 0 ? (g.m - p * g.mstep < g.mmax ? g.m - p * g.mstep : g.mmax) : g.m;
  const int64_t kall = g.mstep > 0 && g.tri == kTriA ? m : g.kk;
  const int64_t lda = g.lda, ldb = g.ldb, ldc = g.ldc, nn = g.nn;
  int64_t R, Cc, kbeg, kk;
  if (!gemm_tile<LOWER, kEb>(g, m, kall, R, Cc, kbeg, kk)) return;  // whole workgroup
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = 32 * (wave >> 1), c0 = 32 * (wave & 1);
  const int lr = lane & 15, lk = lane >> 4;
  f64x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  constexpr int kPer = kEb * kEb / 256;
  double av[kPer], bv[kPer];
  auto load = [&](int64_t kc) {
#pragma unroll
    for (int it = 0; it < kPer; ++it) {
      const int e = (int)threadIdx.x + 256 * it;
      const int x = e / kEb, y = e % kEb;  // consecutive threads: consecutive y
      {
        const int r = TA ? y : x, k = TA ? x : y;
        const bool ok = kc + k < kk && R + r < m;
        av[it] = ok ? (TA ? A[(kc + k) * lda + R + r] : A[(R + r) * lda + kc + k]) : 0.0;
      }
      {
        const int c = TB ? x : y, k = TB ? y : x;
        const bool ok = kc + k < kk && Cc + c < nn;
        bv[it] = ok ? (TB ? B[(Cc + c) * ldb + kc + k] : B[(kc + k) * ldb + Cc + c]) : 0.0;
      }
    }
  };
  auto store = [&]() {
#pragma unroll
    for (int it = 0; it < kPer; ++it) {
      const int e = (int)threadIdx.x + 256 * it;
      const int x = e / kEb, y = e % kEb;
      As[TA ? lds_at<true>(x, y) : lds_at<false>(y, x)] = av[it];
      Bs[TB ? lds_at<false>(y, x) : lds_at<true>(x, y)] = bv[it];
    }
  };
  const int64_t nch = (kk - kbeg + kEb - 1) / kEb;
  const int64_t kfirst = gemm_descends(g.tri) ? kbeg + (nch - 1) * kEb : kbeg;
  const int64_t kstep = gemm_descends(g.tri) ? -kEb : kEb;
  load(kfirst);
  for (int64_t c = 0, kc = kfirst; c < nch; ++c, kc += kstep) {
    if (c > 0) __syncthreads();  // every wave is done with the previous chunk
    store();
    __syncthreads();
    if (c + 1 < nch) load(kc + kstep);
#pragma unroll 4
    for (int k = 0; k < kEb; k += 4) {
      const double a0 = As[lds_at<TA>(k + lk, r0 + lr)], a1 = As[lds_at<TA>(k + lk, r0 + 16 + lr)];
      const double b0 = Bs[lds_at<!TB>(k + lk, c0 + lr)], b1 = Bs[lds_at<!TB>(k + lk, c0 + 16 + lr)];
      acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
    }
  }
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t row = R + r0 + 16 * rb + lk + 4 * i, col = Cc + c0 + 16 * cb + lr;
        if (row < m && col < nn) C[row * ldc + col] = MODE == kNegate ? -acc[rb][cb][i] : acc[rb][cb][i];
      }
}

// The same products in 128 x 128 output tiles, k in chunks of 16 in two LDS
// buffers.
//
// Bound by the FP64 matrix cores (64 cycles per v_mfma_f64_16x16x4 and SIMD,
// 74 TF/s measured on a large library product).  A wave owns a 64 x 64
// quadrant, 16 MFMAs for every 8 operand reads, against 4 for 4 in the 64-wide
// tiles, and a tile reads half the bytes per flop; two workgroups per CU
// (74 KB of LDS each), so one multiplies while the other waits at its barrier.
// Each operand keeps its source orientation in LDS: k-major [k][x], pitch 144
// doubles, or x-major [x][k], pitch 18, both with 16-byte rows and distinct
// banks for the operand reads of a half-wave.  The 16-byte x-major stores do
// conflict (a row spans 32 of 64 banks and the next starts 36 on): 0.5 conflict cycles per
// LDS instruction in L F, 0.9 in the Gram, 1 to 3% of the cycles.  Interior chunks load 16 bytes per
// lane (rows need 8-byte alignment only), edges element by element.
// n = 32,768, r = 4,096: L F takes 9.2 ms (61 TF/s of useful flops; 9.6 with vector
// address arithmetic) against 24 ms in 64-wide tiles over the full square; trailing updates of the exact GP (k = 256)
// reach 39 TF/s against 28.
constexpr int kGt = 128;       // tile edge
constexpr int kGk = 16;        // k per chunk
constexpr int kGKLd = kGt + 16;
constexpr int kGXLd = kGk + 2;
constexpr int64_t kGemmMaxLd = 1 << 22;  // 127 rows within 2^32 bytes
constexpr int kGBuf = kGt * kGXLd > kGk * kGKLd ? kGt * kGXLd : kGk * kGKLd;
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x2u __attribute__((ext_vector_type(2), aligned(8)));

template <bool KMAJOR>
__device__ __forceinline__ int gemm_at(int k, int x) {
  return KMAJOR ? k * kGKLd + x : x * kGXLd + k;
}

// This thread's four 16-byte pieces of the 128 x 16 operand chunks of a tile at x0.
// KMAJOR: element (x, k) at P[k ld + x], otherwise P[x ld + k]; x >= xn reads
// some valid row (its outputs are not stored), k >= kn reads as zero.  A piece's
// address is a scalar pointer to the chunk plus a byte offset within 32 bits (ld <=
// kGemmMaxLd) that the tile fixes, so that a load costs no vector instruction:
// these add to the time of the MFMAs.
template <bool KMAJOR>
struct GemmOperand {
  const double* P;
  int64_t ld, x0, xn, kn;
  uint32_t off[KMAJOR ? 1 : 4];
  __device__ __forceinline__ GemmOperand(const double* P_, int64_t ld_, int64_t x0_, int64_t xn_, int64_t kn_)
      : P(P_), ld(ld_), x0(x0_), xn(xn_), kn(kn_) {
    const int tid = threadIdx.x;
    if constexpr (KMAJOR) {
      off[0] = 8u * ((uint32_t)(tid >> 6) * (uint32_t)ld + 2u * (tid & 63));
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t x = (tid >> 3) + 32 * u;
        off[u] = 8u * ((uint32_t)(x0 + x < xn ? x : xn - 1 - x0) * (uint32_t)ld + 2u * (tid & 7));
      }
    }
  }
  __device__ __forceinline__ void load(int64_t k0, f64x2 (&v)[4]) const {
    if (KMAJOR ? x0 + kGt <= xn && k0 + kGk <= kn : k0 + kGk <= kn) {
      const char* src = (const char*)(KMAJOR ? P + k0 * ld + x0 : P + x0 * ld + k0);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if constexpr (KMAJOR)
          v[u] = *(const f64x2u*)(src + (int64_t)32 * u * ld + off[0]);
        else
          v[u] = *(const f64x2u*)(src + off[u]);
      }
      return;
    }
    const int tid = threadIdx.x;
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        if constexpr (KMAJOR) {
          const int64_t x = x0 + 2 * (tid & 63) + e < xn ? x0 + 2 * (tid & 63) + e : xn - 1;
          const int64_t k = k0 + (tid >> 6) + 4 * u;
          v[u][e] = k < kn ? P[k * ld + x] : 0.0;
        } else {
          const double* src = (const double*)((const char*)(P + x0 * ld + k0) + off[u]);
          v[u][e] = k0 + 2 * (tid & 7) + e < kn ? src[e] : 0.0;
        }
      }
  }
};

template <bool KMAJOR>
__device__ __forceinline__ void gemm_store(double* buf, const f64x2 (&v)[4]) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int at = KMAJOR ? gemm_at<true>((tid >> 6) + 4 * u, 2 * (tid & 63))
                          : gemm_at<false>(2 * (tid & 7), (tid >> 3) + 32 * u);
    *(f64x2*)(buf + at) = v[u];
  }
}

// A(R.., kbeg..kn) B(kbeg..kn, Cc..) of one tile by one workgroup: acc[i][j] is the 16 x 16
// block (i, j) of this wave's quadrant.  nch >= 1 chunks from kfirst in steps of kstep.
template <bool TA, bool TB>
__device__ __forceinline__ void gemm128_mac(const GemmOperand<TA>& opa, const GemmOperand<!TB>& opb, int64_t kfirst,
                                            int64_t kstep, int nch, double (*As)[kGBuf], double (*Bs)[kGBuf],
                                            f64x4 (&acc)[4][4]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = 64 * (wave >> 1), c0 = 64 * (wave & 1);
  const int lr = lane & 15, lk = lane >> 4;
  f64x2 av[4], bv[4];
  opa.load(kfirst, av);
  opb.load(kfirst, bv);
  gemm_store<TA>(As[0], av);
  gemm_store<!TB>(Bs[0], bv);
  __syncthreads();
  int64_t kc = kfirst;
  auto chunk = [&](int c, int cur) {
    const bool more = c + 1 < nch;
    if (more) {
      kc += kstep;
      opa.load(kc, av);
      opb.load(kc, bv);
    }
#pragma unroll
    for (int k = 0; k < kGk; k += 4) {
      double a[4], q[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i] = As[cur][gemm_at<TA>(k + lk, r0 + 16 * i + lr)];
        q[i] = Bs[cur][gemm_at<!TB>(k + lk, c0 + 16 * i + lr)];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], q[j], acc[i][j], 0, 0, 0);
    }
    if (more) {  // the other buffer's readers passed the previous barrier
      gemm_store<TA>(As[cur ^ 1], av);
      gemm_store<!TB>(Bs[cur ^ 1], bv);
    }
    __syncthreads();
  };
  for (int c = 0; c < nch; c += 2) {  // the buffers' addresses are constants
    chunk(c, 0);
    if (c + 1 < nch) chunk(c + 1, 1);
  }
}

template <int MODE>
__device__ __forceinline__ void gemm128_store(double* C, int64_t ldc, int64_t m, int64_t nn, int64_t R, int64_t Cc,
                                              const f64x4 (&acc)[4][4]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = 64 * (wave >> 1), c0 = 64 * (wave & 1);
  const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) {
    double old[4][4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t row = R + r0 + 16 * rb + lk + 4 * i, col = Cc + c0 + 16 * cb + lr;
        old[cb][i] = (MODE == kSubtract && row < m && col < nn) ? C[row * ldc + col] : 0.0;
      }
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t row = R + r0 + 16 * rb + lk + 4 * i, col = Cc + c0 + 16 * cb + lr;
        if (row < m && col < nn)
          C[row * ldc + col] = MODE == kSubtract ? old[cb][i] - acc[rb][cb][i]
                                                 : (MODE == kNegate ? -acc[rb][cb][i] : acc[rb][cb][i]);
      }
  }
}

template <bool TA, bool TB, bool LOWER, int MODE>
__global__ __launch_bounds__(256, 2) void gemm128_f64_kernel(GemmArgs g) {
  __shared__ __attribute__((aligned(16))) double As[2][kGBuf], Bs[2][kGBuf];
  const int64_t p = blockIdx.y;
  const double* __restrict__ A = g.A + p * g.sA;
  const double* __restrict__ B = g.B + p * g.sB;
  double* C = g.C + p * g.sC;
  const int64_t m = g.mstep > 0 ? (g.m - p * g.mstep < g.mmax ? g.m - p * g.mstep : g.mmax) : g.m;
  const int64_t kall = g.mstep > 0 && g.tri == kTriA ? m : g.kk;
  const int64_t ldc = g.ldc, nn = g.nn;
  int64_t R, Cc, kbeg, kn;
  if (!gemm_tile<LOWER, kGt>(g, m, kall, R, Cc, kbeg, kn)) return;  // whole workgroup
  f64x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  const int nch = (int)((kn - kbeg + kGk - 1) / kGk);
  const bool desc = gemm_descends(g.tri);
  gemm128_mac<TA, TB>(GemmOperand<TA>(A, g.lda, R, m, kn), GemmOperand<!TB>(B, g.ldb, Cc, nn, kn),
                      desc ? kbeg + (int64_t)(nch - 1) * kGk : kbeg, desc ? -kGk : kGk, nch, As, Bs, acc);
  gemm128_store<MODE>(C, ldc, m, nn, R, Cc, acc);
}

// C = A A^T over the lower 128-wide tiles (A m x kk), its k range split where the
// tiles alone leave CUs idle: the tiles beyond a multiple of 512 (two workgroups
// per CU) are cut into `parts` runs of k each, whose products go to slabs
// [tile][part][128][128] and are added in the order of k.  m = 4,096, kk = 32,768:
// 528 tiles, of which the last 16 took half as long again as the first 512:
// 13.6 -> 9.4 ms.  m = 1,024, kk = 8,192: 0.45 ms in 64-wide
// tiles, 0.22 so.
struct GramSplit {
  int64_t full;  // tiles computed whole
  int rest, parts;
};

__global__ __launch_bounds__(256, 2) void gram128_f64_kernel(GemmArgs g, GramSplit gs, double* slab) {
  __shared__ __attribute__((aligned(16))) double As[2][kGBuf], Bs[2][kGBuf];
  const int64_t h = blockIdx.x;
  int64_t b, slot = -1;
  int c0 = 0, c1 = (int)((g.kk + kGk - 1) / kGk);
  if (h < gs.full) {  // as in gemm_tile, each XCD a contiguous run
    const int64_t xcd = h & 7, q8 = gs.full >> 3, rem8 = gs.full & 7;
    b = xcd * q8 + (xcd < rem8 ? xcd : rem8) + (h >> 3);
  } else {
    slot = h - gs.full;
    b = gs.full + slot / gs.parts;
    const int part = (int)(slot % gs.parts), n = c1;
    c0 = (int)((int64_t)n * part / gs.parts);
    c1 = (int)((int64_t)n * (part + 1) / gs.parts);
  }
  int64_t ti, tj;
  lower_tile(b, ti, tj);
  const int64_t R = kGt * ti, Cc = kGt * tj;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  f64x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  gemm128_mac<false, true>(GemmOperand<false>(g.A, g.lda, R, g.m, g.kk), GemmOperand<false>(g.A, g.lda, Cc, g.m, g.kk),
                           (int64_t)c0 * kGk, kGk, c1 - c0, As, Bs, acc);
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 64 * (wave >> 1) + 16 * rb + lk + 4 * i, c = 64 * (wave & 1) + 16 * cb + lr;
        if (slot >= 0)
          slab[slot * (kGt * kGt) + r * kGt + c] = acc[rb][cb][i];
        else if (R + r < g.m && Cc + c < g.m)
          g.C[(R + r) * g.ldc + Cc + c] = acc[rb][cb][i];
      }
}

// The split tiles' sums.  grid = (64, rest).
__global__ __launch_bounds__(256) void gram_slab_sum_kernel(GemmArgs g, GramSplit gs, const double* __restrict__ slab) {
  const int64_t b = gs.full + blockIdx.y;
  int64_t ti, tj;
  lower_tile(b, ti, tj);
  const int e = blockIdx.x * 256 + threadIdx.x;
  const int64_t row = kGt * ti + e / kGt, col = kGt * tj + e % kGt;
  if (row >= g.m || col >= g.m) return;
  const double* src = slab + (int64_t)blockIdx.y * gs.parts * (kGt * kGt) + e;
  double s = 0.0;
  int p = 0;
  for (; p + 8 <= gs.parts; p += 8) {
    double v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = src[(int64_t)(p + j) * (kGt * kGt)];
#pragma unroll
    for (int j = 0; j < 8; ++j) s += v[j];
  }
  for (; p < gs.parts; ++p) s += src[(int64_t)p * (kGt * kGt)];
  g.C[row * g.ldc + col] = s;
}

static int64_t tile_count(bool lower, int64_t m, int64_t nn, int64_t edge) {
  const int64_t nrt = (m + edge - 1) / edge, nct = (nn + edge - 1) / edge;
  return lower ? nrt * (nrt + 1) / 2 : nrt * nct;
}

// The 128-wide tiles fill the chip from about this many on; below it the
// 64-wide tiles, four times as many, use more of the 256 CUs.
constexpr int64_t kGemm128MinTiles = 256;

static bool use_gemm128(bool lower, int64_t m, int64_t nn) { return tile_count(lower, m, nn, kGt) >= kGemm128MinTiles; }

// `batch` products (blockIdx.y); g.nrt and g.nct are filled in here.  g.mmax rows per batch when batched.
template <bool TA, bool TB, bool LOWER, int MODE, bool WIDE>
static hipError_t gemm_launch(GemmArgs g, int64_t batch, hipStream_t st) {
  constexpr int64_t edge = WIDE ? kGt : kEb;
  const int64_t rows = g.mstep > 0 ? g.mmax : g.m;
  const int64_t tiles = tile_count(LOWER, rows, g.nn, edge);
  if (tiles <= 0 || batch <= 0) return hipSuccess;
  if (tiles > 0x7fffffff || batch > 65535 || g.kk < 1) return hipErrorInvalidValue;
  if constexpr (WIDE)
    if (g.lda > kGemmMaxLd || g.ldb > kGemmMaxLd) return gemm_launch<TA, TB, LOWER, MODE, false>(g, batch, st);
  g.nrt = (int)((rows + edge - 1) / edge);
  g.nct = (int)((g.nn + edge - 1) / edge);
  const dim3 grid((unsigned)tiles, (unsigned)batch);
  if constexpr (WIDE)
    gemm128_f64_kernel<TA, TB, LOWER, MODE><<<grid, 256, 0, st>>>(g);
  else
    gemm64_f64_kernel<TA, TB, LOWER, MODE><<<grid, 256, 0, st>>>(g);
  return hipGetLastError();
}

static int ntiles(int64_t len) { return (int)((len + kEb - 1) / kEb); }

// Workgroup 0 factors the 64-wide diagonal block at j0; the others take tiles
// [t0, t0 + gridDim.x - 1) of the lower 128-wide tiles of A[j2.., j2..] -= P P^T, P =
// A[j2.., p0 .. p0 + kb): the trailing update left by the super-panel before.  The
// two touch different parts of A (j0 + 64 <= j2, p0 + kb <= j0).
__global__ __launch_bounds__(256, 2) void potrf_update_kernel(double* A, int64_t n, int64_t j0, int jb, int* info,
                                                              double* Dinv, int64_t j2, int64_t p0, int kb,
                                                              int64_t t0) {
  constexpr int kPotrf = 2 * kEb * kDbLd, kGemm = 4 * kGBuf;
  __shared__ __attribute__((aligned(16))) double sh[kPotrf > kGemm ? kPotrf : kGemm];
  if (blockIdx.x == 0) {
    potrf_diag(A, n, j0, jb, info, Dinv, sh, sh + kEb * kDbLd);
    return;
  }
  // each XCD takes a contiguous run of the tiles
  const int64_t T = gridDim.x - 1, h = blockIdx.x - 1, xcd = h & 7, q8 = T >> 3, rem8 = T & 7;
  int64_t ti, tj;
  lower_tile(t0 + xcd * q8 + (xcd < rem8 ? xcd : rem8) + (h >> 3), ti, tj);
  const int64_t m = n - j2, R = kGt * ti, Cc = kGt * tj;
  const double* P = A + j2 * n + p0;
  f64x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  gemm128_mac<false, true>(GemmOperand<false>(P, n, R, m, kb), GemmOperand<false>(P, n, Cc, m, kb), 0, kGk,
                           (kb + kGk - 1) / kGk, (double(*)[kGBuf])sh, (double(*)[kGBuf])(sh + 2 * kGBuf), acc);
  gemm128_store<kSubtract>(A + j2 * n + j2, n, m, m, R, Cc, acc);
}

// A = L L^T in place (lower triangle; the diagonal blocks' upper parts are
// zeroed, the rest of the upper triangle holds no result); the inverses of the
// diagonal blocks stay in Dinv (block bi at 64 * 64 * bi).  Two levels of
// blocking: 64-wide panels inside 256-wide super-panels.  A panel updates only
// the columns of its own super-panel; what lies beyond takes the whole super-panel
// at once (k = 256), so that it is read and written once per 256 columns instead
// of once per 64: first the next super-panel's columns, and the rest beside the next
// four diagonal blocks, each of which is 31 to 35 us of one workgroup: up to 255 tiles, one per
// CU (50 us), beside each block, in as few launches as that allows; more per launch only
// where four launches do not hold them.  n = 7,503: 10.3 ms with the trailing update in
// launches of its own and the panel's own updates in two, 8.9 ms so (17.5 instead of
// 19.1 ms for value, gradient and inverse); four equal shares, each with
// a tile's 50 us: 9.8 ms.
constexpr int kSp = 4 * kEb;

static hipError_t cholesky(double* A, int64_t n, int* info, double* Dinv, hipStream_t st) {
  if (n > kGemmMaxLd) return hipErrorInvalidValue;  // 2^47 bytes
  hipError_t e = hipSuccess;
  for (int64_t J0 = 0; J0 < n; J0 += kSp) {
    const int64_t Jend = std::min<int64_t>(n, J0 + kSp);
    // the trailing update by the super-panel before this one, columns from Jend on
    const int64_t shared = J0 > 0 ? tile_count(true, n - Jend, n - Jend, kGt) : 0;
    const int64_t per = std::max<int64_t>(255, (shared + 3) / 4);
    for (int64_t j0 = J0; j0 < Jend; j0 += kEb) {
      const int jb = (int)std::min<int64_t>(kEb, n - j0);
      const int64_t rest = n - j0 - jb, q = (j0 - J0) / kEb;
      double* Di = Dinv + j0 / kEb * kEb * kEb;
      const int64_t t0 = std::min(shared, q * per), t1 = std::min(shared, (q + 1) * per);
      potrf_update_kernel<<<(unsigned)(1 + t1 - t0), 256, 0, st>>>(A, n, j0, jb, info, Di, Jend, J0 - kSp, kSp, t0);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      if (rest <= 0) return hipSuccess;
      // L21 = A21 L11^{-T} for every row below (jb = 64 here)
      e = tile_update<false, true>(A, n, j0, Di, kEb, 0, 0, A, n, jb, j0 + jb, j0, ntiles(rest), 1, st);
      if (e != hipSuccess) return e;
      // the rest of this super-panel's columns, [j0 + 64, Jend), on and below the diagonal
      const int64_t wcols = Jend - j0 - jb;
      if (wcols > 0) {
        e = tile_update<true, false>(A, n, j0, A, n, -1, j0, A, n, jb, j0 + jb, j0 + jb, ntiles(rest), ntiles(wcols), st);
        if (e != hipSuccess) return e;
      }
    }
    // the next super-panel's columns, k = 256
    if (n > Jend) {
      e = tile_update<true, false>(A, n, J0, A, n, -1, J0, A, n, kSp, Jend, Jend, ntiles(n - Jend),
                                   ntiles(std::min<int64_t>(kSp, n - Jend)), st);
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

// ---------------------------------------------------------------- K_hat^{-1}

// The diagonal blocks of the factor replaced by their inverses, the upper half
// of every 128-wide diagonal tile zeroed; dL (nullable) receives the factor's
// diagonal.  One workgroup per 64-row block.
__global__ __launch_bounds__(256) void seed_inverse_kernel(double* __restrict__ A, int64_t n,
                                                           const double* __restrict__ Dinv, double* __restrict__ dL) {
  const int64_t bi = blockIdx.x, i0 = bi * kEb;
  if (dL && threadIdx.x < kEb && i0 + threadIdx.x < n)
    dL[i0 + threadIdx.x] = A[(i0 + threadIdx.x) * n + i0 + threadIdx.x];
  __syncthreads();
  for (int e = threadIdx.x; e < kEb * kEb; e += 256) {
    const int64_t r = i0 + e / kEb, c = i0 + e % kEb;
    if (r < n && c < n) A[r * n + c] = Dinv[bi * kEb * kEb + e];
    if ((bi & 1) == 0 && r < n && c + kEb < n) A[r * n + c + kEb] = 0.0;
  }
}

// A <- L^{-1} in place (lower triangle; zero above the diagonal inside the
// 128-wide diagonal tiles, nothing beyond them) from the factor L in A and its
// diagonal blocks' inverses; W is scratch of the same size.  Doubling: with the
// inverses X of the size-s diagonal blocks in place, each pair of neighbours
// takes X21 = -X22 (L21 X11), all pairs of a size in two launches, so the work
// is ~log2(n / 64) large triangular products instead of a sweep of 64-row
// steps that rewrites the trailing rows for each.
static hipError_t lower_inverse(double* A, double* W, const double* Dinv, double* dL, int64_t n, hipStream_t st) {
  seed_inverse_kernel<<<(unsigned)((n + kEb - 1) / kEb), 256, 0, st>>>(A, n, Dinv, dL);
  hipError_t e = hipGetLastError();
  for (int64_t s = kEb; s < n && e == hipSuccess; s *= 2) {
    const int64_t pairs = (n - s + 2 * s - 1) / (2 * s);  // blocks p with a row beyond (2 p + 1) s
    const int64_t step = 2 * s * (n + 1);
    double* L21 = A + s * n;
    // W21 = L21 X11, then A21 = -X22 W21
    const GemmArgs t{L21, n, step, A, n, step, W + s * n, n, step, n - s, s, s, s, 2 * s, 0, 0, kTriB};
    const GemmArgs x{A + s * (n + 1), n, step, W + s * n, n, step, L21, n, step, n - s, s, s, s, 2 * s, 0, 0, kTriA};
    if (tile_count(false, s, s, kGt) * pairs >= kGemm128MinTiles) {
      e = gemm_launch<false, false, false, kAssign, true>(t, pairs, st);
      if (e == hipSuccess) e = gemm_launch<false, false, false, kNegate, true>(x, pairs, st);
    } else {
      e = gemm_launch<false, false, false, kAssign, false>(t, pairs, st);
      if (e == hipSuccess) e = gemm_launch<false, false, false, kNegate, false>(x, pairs, st);
    }
  }
  return e;
}

// The lower tiles of B = K_hat^{-1} = X^T X, X = L^{-1} left in A.
static hipError_t inverse_from_cholesky(double* A, double* B, const double* Dinv, double* dL, int64_t n,
                                        hipStream_t st) {
  hipError_t e = lower_inverse(A, B, Dinv, dL, n, st);
  if (e != hipSuccess) return e;
  const GemmArgs g{A, n, 0, A, n, 0, B, n, 0, n, n, n, 0, 0, 0, 0, kTriAt};
  return use_gemm128(true, n, n) ? gemm_launch<true, false, true, kAssign, true>(g, 1, st)
                                 : gemm_launch<true, false, true, kAssign, false>(g, 1, st);
}

// B[r][c] = B[c][r] for c > r (the upper triangle from the lower one).
__global__ void mirror_kernel(double* __restrict__ B, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * n) return;
  const int64_t r = e / n, c = e - r * n;
  if (c > r) B[e] = B[c * n + r];
}

// out[a] = sum_b B[a][b] v[b], one wave per row (fixed summation order).
__global__ __launch_bounds__(256) void gemv_rows_kernel(const double* __restrict__ B, const double* __restrict__ v,
                                                        int64_t n, double* __restrict__ out) {
  const int64_t a = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
  const int lane = threadIdx.x % 64;
  if (a >= n) return;
  double s = 0.0;
  for (int64_t b = lane; b < n; b += 64) s = fma(B[a * n + b], v[b], s);
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (lane == 0) out[a] = s;
}

__global__ void diag_kernel(const double* __restrict__ B, int64_t n, double* __restrict__ dB) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dB[i] = B[i * n + i];
}

// ---------------------------------------------------------------- gradient

// Per lower tile (a >= b): partial sums over its pairs of
//   w M_ab psi_ab (x~_aj - x~_bj)^2   (j < d)   and   w M_ab k_ab   (entry d),
// M = omega omega^T - K_hat^{-1}, w = 2 below the diagonal and 1 on it,
// x~ = x / l.  One partial row of DP + 1 per tile.
template <int KIND, int DP>
__global__ __launch_bounds__(256) void exact_grad_kernel(const double* __restrict__ X, int64_t n, int d,
                                                         const double* __restrict__ il, double sf,
                                                         const double* __restrict__ Kinv,
                                                         const double* __restrict__ om,
                                                         double* __restrict__ partial) {
  __shared__ double xa[kEb][DP];   // rows of a tile are wave-uniform: broadcast reads
  __shared__ double xbT[DP][kEb];
  double(*red)[DP + 1] = reinterpret_cast<double(*)[DP + 1]>(&xa[0][0]);  // after the pair loop only
  const int64_t b = blockIdx.x;
  int64_t ti = (int64_t)((sqrt(8.0 * (double)b + 1.0) - 1.0) * 0.5);
  while ((ti + 1) * (ti + 2) / 2 <= b) ++ti;
  while (ti * (ti + 1) / 2 > b) --ti;
  const int64_t tj = b - ti * (ti + 1) / 2;
  const int64_t a0 = ti * kEb, b0 = tj * kEb;
  for (int e = threadIdx.x; e < kEb * DP; e += 256) {
    const int row = e / DP, f = e % DP;
    const bool fin = f < d;
    xa[row][f] = (a0 + row < n && fin) ? X[(a0 + row) * d + f] * il[f] : 0.0;
    xbT[f][row] = (b0 + row < n && fin) ? X[(b0 + row) * d + f] * il[f] : 0.0;
  }
  __syncthreads();
  const int c = threadIdx.x % kEb, rb = threadIdx.x / kEb;
  double acc[DP + 1];
#pragma unroll
  for (int f = 0; f <= DP; ++f) acc[f] = 0.0;
  const int64_t bb = b0 + c;
  if (bb < n) {
    const double ob = om[bb];
    for (int j = 0; j < 16; ++j) {
      const int r = rb + 4 * j;
      const int64_t aa = a0 + r;
      if (aa >= n || aa < bb) continue;
      double r2 = 0.0;
#pragma unroll
      for (int f = 0; f < DP; ++f) {
        const double t = xa[r][f] - xbT[f][c];
        r2 = fma(t, t, r2);
      }
      double k, psi;
      if constexpr (KIND == GP_MATERN52) {
        const double u = sqrt(5.0 * r2);
        const double e = exp(-u);
        k = sf * (1.0 + u + u * u / 3.0) * e;
        psi = (5.0 / 3.0) * sf * (1.0 + u) * e;
      } else {
        k = sf * exp(-0.5 * r2);
        psi = k;
      }
      const double w = (aa == bb ? 1.0 : 2.0) * (om[aa] * ob - Kinv[aa * n + bb]);
      const double wp = w * psi;
#pragma unroll
      for (int f = 0; f < DP; ++f) {
        const double t = xa[r][f] - xbT[f][c];
        acc[f] = fma(wp * t, t, acc[f]);
      }
      acc[DP] = fma(w, k, acc[DP]);
    }
  }
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
#pragma unroll
  for (int f = 0; f <= DP; ++f)
    for (int o = 32; o > 0; o >>= 1) acc[f] += __shfl_xor(acc[f], o);
  __syncthreads();  // every wave is done with xa before it becomes the reduction rows
  if (lane == 0) {
#pragma unroll
    for (int f = 0; f <= DP; ++f) red[wave][f] = acc[f];
  }
  __syncthreads();
  for (int f = threadIdx.x; f <= DP; f += 256)
    partial[b * (DP + 1) + f] = ((red[0][f] + red[1][f]) + red[2][f]) + red[3][f];
}

// out[f] = sum over units of partial[u][f], f <= dp, in unit order.
__global__ void sum_units_kernel(const double* __restrict__ partial, int64_t units, int dp1,
                                 double* __restrict__ out) {
  const int f = blockIdx.x;
  __shared__ double s[256];
  double v = 0.0;
  for (int64_t u = threadIdx.x; u < units; u += 256) v += partial[u * dp1 + f];
  s[threadIdx.x] = v;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) s[threadIdx.x] += s[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[f] = s[0];
}

static int exact_dp(int d) { return d <= 16 ? 16 : d <= 32 ? 32 : d <= 48 ? 48 : 64; }

template <int KIND>
static hipError_t launch_exact_grad(int dp, unsigned tiles, const double* X, int64_t n, int d, const double* il,
                                    double sf, const double* Kinv, const double* om, double* partial,
                                    hipStream_t st) {
  switch (dp) {
    case 16: exact_grad_kernel<KIND, 16><<<tiles, 256, 0, st>>>(X, n, d, il, sf, Kinv, om, partial); break;
    case 32: exact_grad_kernel<KIND, 32><<<tiles, 256, 0, st>>>(X, n, d, il, sf, Kinv, om, partial); break;
    case 48: exact_grad_kernel<KIND, 48><<<tiles, 256, 0, st>>>(X, n, d, il, sf, Kinv, om, partial); break;
    default: exact_grad_kernel<KIND, 64><<<tiles, 256, 0, st>>>(X, n, d, il, sf, Kinv, om, partial); break;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------- driver

static int64_t lower_tiles(int64_t n) {
  const int64_t t = (n + kEb - 1) / kEb;
  return t * (t + 1) / 2;
}

size_t exact_ws_bytes(int d, int64_t n) {
  if (n < 1 || n > kExactMaxN || d < 1 || d > kExactMaxD) return 0;
  size_t b = 2 * align256((size_t)n * n * 8);                            // K_hat -> L -> L^{-1}; scratch -> K_hat^{-1}
  b += 3 * align256((size_t)n * 8);                                      // omega, diag L, diag K_hat^{-1}
  b += 2 * align256((size_t)GP_MAX_D * 8);                               // feature scales
  b += align256((size_t)lower_tiles(n) * (exact_dp(d) + 1) * 8);         // gradient partials
  b += align256((size_t)(kExactMaxD + 1) * 8) + align256(sizeof(int));   // sums, info
  b += align256((size_t)((n + kEb - 1) / kEb) * kEb * kEb * 8);          // diagonal-block inverses
  return b + 4096;
}

int run_exact(const gp_kernel* kern, const double* X, const double* y, int64_t n, double* mll, double* grad,
              double* omega_out, void* ws, size_t ws_bytes, hipStream_t st) {
  const int d = kern->d;
  const int dp = exact_dp(d);
  Carve cv(ws, ws_bytes);
  double* A = cv.take<double>((size_t)n * n);
  double* B = cv.take<double>((size_t)n * n);
  double* om = cv.take<double>(n);
  double* dA = cv.take<double>(n);
  double* dB = cv.take<double>(n);
  double* sc = cv.take<double>(GP_MAX_D);
  double* il = cv.take<double>(GP_MAX_D);
  const int64_t tiles = lower_tiles(n);
  double* part = cv.take<double>((size_t)tiles * (dp + 1));
  double* sums = cv.take<double>(kExactMaxD + 1);
  int* info = cv.take<int>(1);
  double* Dinv = cv.take<double>((size_t)((n + kEb - 1) / kEb) * kEb * kEb);
  if (!Dinv) return fail(GP_EWORKSPACE, "gp_exact_mll_and_grad: workspace layout failed");
  std::vector<double> h_sc(d), h_il(d);
  for (int f = 0; f < d; ++f) {
    h_il[f] = 1.0 / kern->lengthscale[f];
    h_sc[f] = (kern->kind == GP_MATERN52 ? std::sqrt(5.0) : 1.0) * h_il[f];
  }
  const int zero = 0;
  GPK_HIP(hipMemcpyAsync(sc, h_sc.data(), sizeof(double) * d, hipMemcpyHostToDevice, st));
  GPK_HIP(hipMemcpyAsync(il, h_il.data(), sizeof(double) * d, hipMemcpyHostToDevice, st));
  GPK_HIP(hipMemcpyAsync(info, &zero, sizeof(int), hipMemcpyHostToDevice, st));
  const dim3 g2((unsigned)ntiles(n), (unsigned)ntiles(n));
  if (kern->kind == GP_MATERN52)
    form_khat_kernel<GP_MATERN52><<<g2, 256, 0, st>>>(X, n, d, sc, kern->outputscale, kern->noise, A);
  else
    form_khat_kernel<GP_RBF><<<g2, 256, 0, st>>>(X, n, d, sc, kern->outputscale, kern->noise, A);
  GPK_HIP(hipGetLastError());
  GPK_HIP(cholesky(A, n, info, Dinv, st));
  GPK_HIP(inverse_from_cholesky(A, B, Dinv, dA, n, st));
  mirror_kernel<<<(unsigned)((n * n + 255) / 256), 256, 0, st>>>(B, n);
  GPK_HIP(hipGetLastError());
  gemv_rows_kernel<<<(unsigned)((n + 3) / 4), 256, 0, st>>>(B, y, n, om);
  GPK_HIP(hipGetLastError());
  diag_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(B, n, dB);
  GPK_HIP(hipGetLastError());
  if (grad) {
    if (kern->kind == GP_MATERN52)
      GPK_HIP(launch_exact_grad<GP_MATERN52>(dp, (unsigned)tiles, X, n, d, il, kern->outputscale, B, om, part, st));
    else
      GPK_HIP(launch_exact_grad<GP_RBF>(dp, (unsigned)tiles, X, n, d, il, kern->outputscale, B, om, part, st));
    sum_units_kernel<<<(unsigned)(dp + 1), 256, 0, st>>>(part, tiles, dp + 1, sums);
    GPK_HIP(hipGetLastError());
  }
  std::vector<double> h_om(n), h_dA(n), h_dB(n), h_y(n), h_sums(dp + 1);
  int h_info = 0;
  GPK_HIP(hipMemcpyAsync(h_om.data(), om, sizeof(double) * n, hipMemcpyDeviceToHost, st));
  GPK_HIP(hipMemcpyAsync(h_dA.data(), dA, sizeof(double) * n, hipMemcpyDeviceToHost, st));
  GPK_HIP(hipMemcpyAsync(h_dB.data(), dB, sizeof(double) * n, hipMemcpyDeviceToHost, st));
  GPK_HIP(hipMemcpyAsync(h_y.data(), y, sizeof(double) * n, hipMemcpyDeviceToHost, st));
  if (grad) GPK_HIP(hipMemcpyAsync(h_sums.data(), sums, sizeof(double) * (dp + 1), hipMemcpyDeviceToHost, st));
  GPK_HIP(hipMemcpyAsync(&h_info, info, sizeof(int), hipMemcpyDeviceToHost, st));
  if (omega_out) GPK_HIP(hipMemcpyAsync(omega_out, om, sizeof(double) * n, hipMemcpyDeviceToDevice, st));
  GPK_HIP(hipStreamSynchronize(st));
  if (h_info != 0)
    return fail(GP_ENOTPD, "gp_exact_mll_and_grad: K_hat is not numerically positive definite (pivot %d)", h_info - 1);
  double quad = 0.0, logdet = 0.0, wtw = 0.0, tr = 0.0;
  for (int64_t i = 0; i < n; ++i) {
    quad += h_y[i] * h_om[i];
    logdet += 2.0 * std::log(h_dA[i]);
    wtw += h_om[i] * h_om[i];
    tr += h_dB[i];
  }
  const double v = -0.5 * quad - 0.5 * logdet - 0.5 * (double)n * std::log(2.0 * M_PI);
  if (!std::isfinite(v)) return fail(GP_ENONFINITE, "gp_exact_mll_and_grad: non-finite log marginal likelihood");
  *mll = v;
  if (grad) {
    for (int j = 0; j < d; ++j) grad[j] = 0.5 * h_sums[j];
    grad[d] = 0.5 * h_sums[dp];
    grad[d + 1] = 0.5 * kern->noise * (wtw - tr);
    for (int j = 0; j < d + 2; ++j)
      if (!std::isfinite(grad[j])) return fail(GP_ENONFINITE, "gp_exact_mll_and_grad: non-finite gradient");
  }
  return GP_OK;
}

// ---------------------------------------------------------------- exported dense pieces

hipError_t dense_lower_times(int64_t m, int64_t nn, const double* L, int64_t ldl, const double* B, int64_t ldb,
                             double* C, int64_t ldc, hipStream_t st) {
  const GemmArgs g{L, ldl, 0, B, ldb, 0, C, ldc, 0, m, nn, m, 0, 0, 0, 0, kTriA};
  return use_gemm128(false, m, nn) ? gemm_launch<false, false, false, kAssign, true>(g, 1, st)
                                   : gemm_launch<false, false, false, kAssign, false>(g, 1, st);
}

// The split that ends soonest: 512 workgroups run at a time, up to 256 of a last
// round at twice the speed; a part has at least 16 chunks of k, and the slabs
// fit the scratch memory.
static GramSplit gram_split(int64_t tiles, int64_t kk, int64_t scratch_doubles) {
  GramSplit gs{tiles, 0, 1};
  const int64_t rest = tiles % 512;
  if (rest == 0) return gs;
  const int64_t cap = std::min((kk + kGk - 1) / kGk / 16, scratch_doubles / (rest * kGt * kGt));
  double best = 1e300;
  int parts = 1;
  for (int64_t p = 1; p <= std::max<int64_t>(1, std::min<int64_t>(cap, 512)); ++p) {
    const int64_t items = rest * p, last = items % 512;
    const double t = ((double)(items / 512) + (last == 0 ? 0.0 : last <= 256 ? 0.5 : 1.0)) / (double)p;
    if (t < 0.98 * best) {
      best = t;
      parts = (int)p;
    }
  }
  if (parts > 1) gs = GramSplit{tiles - rest, (int)rest, parts};
  return gs;
}

hipError_t dense_gram(int64_t m, int64_t kk, const double* A, int64_t lda, double* C, int64_t ldc, double* scratch,
                      int64_t scratch_doubles, hipStream_t st) {
  if (m < 1 || kk < 1) return hipErrorInvalidValue;
  const GemmArgs g{A, lda, 0, A, lda, 0, C, ldc, 0, m, m, kk, 0, 0, 0, 0, kTriNone};
  const int64_t tiles = tile_count(true, m, m, kGt);
  const GramSplit gs = gram_split(tiles, kk, scratch_doubles);
  if (lda > kGemmMaxLd || (gs.rest == 0 && !use_gemm128(true, m, m)))
    return gemm_launch<false, true, true, kAssign, false>(g, 1, st);
  const int64_t items = gs.full + (int64_t)gs.rest * gs.parts;
  if (items > 0x7fffffff) return hipErrorInvalidValue;
  gram128_f64_kernel<<<(unsigned)items, 256, 0, st>>>(g, gs, scratch);
  if (gs.rest > 0) gram_slab_sum_kernel<<<dim3(kGt * kGt / 256, (unsigned)gs.rest), 256, 0, st>>>(g, gs, scratch);
  return hipGetLastError();
}

size_t dense_dinv_doubles(int64_t n) { return (size_t)((n + kEb - 1) / kEb) * kEb * kEb; }

hipError_t dense_cholesky(double* A, int64_t n, int* info, double* Dinv, hipStream_t st) {
  return cholesky(A, n, info, Dinv, st);
}

hipError_t dense_lower_inverse(double* L, double* W, const double* Dinv, int64_t n, hipStream_t st) {
  return lower_inverse(L, W, Dinv, nullptr, n, st);
}

}  // namespace gpk

using namespace gpk;

extern "C" int gp_exact_mll_and_grad(const gp_kernel* kern, const double* X, const double* y, int64_t n, double* mll,
                                     double* grad, double* omega, void* ws, size_t ws_bytes, void* stream) {
  GPK_TRY(check_kernel(kern));
  if (!X || !y || !mll) return fail(GP_EINVAL, "gp_exact_mll_and_grad: NULL argument");
  if (n < 1 || n > kExactMaxN) return fail(GP_EINVAL, "gp_exact_mll_and_grad: n=%lld outside [1, %lld]", (long long)n,
                                           (long long)kExactMaxN);
  if (kern->d > kExactMaxD) return fail(GP_EINVAL, "gp_exact_mll_and_grad: d=%d above %d", kern->d, kExactMaxD);
  GPK_TRY(check_ws(ws, ws_bytes, exact_ws_bytes(kern->d, n), "gp_exact_mll_and_grad"));
  return run_exact(kern, X, y, n, mll, grad, omega, ws, ws_bytes, (hipStream_t)stream);
}
