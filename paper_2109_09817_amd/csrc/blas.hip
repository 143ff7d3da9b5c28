// FP64 kernels of the solver: column reductions, the mBCG recurrences, the
// pivoted-Cholesky preconditioner (build and Woodbury apply) and the probe
// generator.  These passes stream O(n s) or O(n k) data per call and are
// bound by HBM bandwidth; all reductions are two-pass with a fixed order
// (per-block partials, then one block per output), so results are bitwise
// reproducible run to run.
//
// Layout: every block of vectors is column-major with leading dimension n
// (column c of an n x s block starts at c*n).
#include "reduce.h"
#include "solver.h"

namespace gpk {

constexpr int kThreads = 256;

// partial[blk * s + c] = sum over this block's rows of A[c*n+i] * B[c*n+i].
// grid = (nblk, s).  Rows are split in contiguous ranges per block.
__global__ void coldot_partial_kernel(const double* __restrict__ A, const double* __restrict__ B, int64_t n,
                                      int64_t rows_per_blk, int s, double* __restrict__ partial) {
  __shared__ double sh[kThreads / 64];
  const int c = blockIdx.y;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_blk;
  const int64_t r1 = r0 + rows_per_blk < n ? r0 + rows_per_blk : n;
  const double* a = A + (int64_t)c * n;
  const double* b = B + (int64_t)c * n;
  double acc = 0.0;
  for (int64_t i = r0 + threadIdx.x; i < r1; i += blockDim.x) acc += a[i] * b[i];
  const double r = block_sum(acc, sh);
  if (threadIdx.x == 0) partial[(int64_t)blockIdx.x * s + c] = r;
}

// out[c] = sum_blk partial[blk * s + c] (fixed order).  grid = (s).
__global__ void reduce_partials_kernel(const double* __restrict__ partial, int64_t nblk, int s,
                                       double* __restrict__ out) {
  __shared__ double sh[kThreads / 64];
  const int c = blockIdx.x;
  double acc = 0.0;
  for (int64_t b = threadIdx.x; b < nblk; b += blockDim.x) acc += partial[b * s + c];
  const double r = block_sum(acc, sh);
  if (threadIdx.x == 0) out[c] = r;
}

// ------------------------------------------------------------------ mBCG steps

// An iteration's scalars are formed where they are used: every workgroup of a
// column adds that column's partial sums itself, all in the same order, so the
// step sizes need no launches of their own.  An iteration at n = 2,048 is bound by
// its launches: 10 now and one copy to the host, 15 and two before (a likelihood
// with 9 iterations and 20 pivots: 2.00 -> 1.54 ms).  Where there are many partial
// sums they are added once before (kSumInPlace).  gamma and active have two copies, read
// from one and written to the other, since workgroups of a column do not run in
// step; the column's first workgroup stores them and the host's records.

// sum_b partial[b * s + c] for every thread of the block, added as by reduce_partials_kernel.
__device__ __forceinline__ double column_sum(const double* __restrict__ partial, int64_t nblk, int s, int c, double* sh,
                                             double* bc) {
  double acc = 0.0;
  for (int64_t b = threadIdx.x; b < nblk; b += blockDim.x) acc += partial[b * s + c];
  const double r = block_sum(acc, sh);
  if (threadIdx.x == 0) *bc = r;
  __syncthreads();
  return *bc;
}

// alpha = gamma / (d.w) for active columns (0 for frozen ones), flagging breakdown;
// U += alpha D ; R -= alpha W ; rpart ||R||^2.  grid = (nblk, s).
__global__ __launch_bounds__(kThreads) void mbcg_update_ur_kernel(MbcgState st, int cur, int64_t nblk,
                                                                  const double* __restrict__ D,
                                                                  const double* __restrict__ W, double* __restrict__ U,
                                                                  double* __restrict__ R, int64_t n,
                                                                  int64_t rows_per_blk) {
  __shared__ double sh[kThreads / 64], bc;
  const int c = blockIdx.y;
  const double dl = column_sum(st.dpart, nblk, st.s, c, sh, &bc);
  const double gamma = st.gamma[cur][c];
  double a = 0.0;
  unsigned flag = 0;
  if (st.active[cur][c]) {
    if (!isfinite(dl) || !isfinite(gamma))
      flag = kStatusNonFinite;
    else if (!(dl > 0.0))
      flag = kStatusNotPD;
    else
      a = gamma / dl;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (flag) atomicOr(st.status, flag);
    st.alpha[c] = a;
  }
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_blk;
  const int64_t r1 = r0 + rows_per_blk < n ? r0 + rows_per_blk : n;
  const int64_t off = (int64_t)c * n;
  double acc = 0.0;
  for (int64_t i = r0 + threadIdx.x; i < r1; i += blockDim.x) {
    const double r = R[off + i] - a * W[off + i];
    U[off + i] += a * D[off + i];
    R[off + i] = r;
    acc += r * r;
  }
  const double s = block_sum(acc, sh);
  if (threadIdx.x == 0) st.rpart[(int64_t)blockIdx.x * st.s + c] = s;
}

// Convergence bookkeeping of iteration j (from rpart), beta = gamma'/gamma (from
// gpart) for columns still active (0 for frozen ones), and D = Z + beta D for
// active columns, 0 for frozen ones.  grid = (nblk, s).
__global__ __launch_bounds__(kThreads) void mbcg_update_d_kernel(MbcgState st, int cur, int64_t nblk, int j, double tol,
                                                                 const double* __restrict__ Z, double* __restrict__ D,
                                                                 int64_t n, int64_t rows_per_blk) {
  __shared__ double sh[kThreads / 64], bc;
  const int c = blockIdx.y;
  const bool was = st.active[cur][c] != 0;
  double b = 0.0, gamma = st.gamma[cur][c], rn = 0.0;
  bool act = was;
  if (was) {  // the same for the whole block
    const double bnorm = st.bnorm[c];
    rn = sqrt(column_sum(st.rpart, nblk, st.s, c, sh, &bc));
    act = !(rn <= tol * bnorm);
    __syncthreads();  // bc is written again
    if (act) {
      const double gn = column_sum(st.gpart, nblk, st.s, c, sh, &bc);
      b = gn / gamma;
      gamma = gn;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (was) {
      st.iters[c] = j + 1;
      st.relres[c] = st.bnorm[c] > 0.0 ? rn / st.bnorm[c] : 0.0;
      if (!isfinite(rn) || (act && !isfinite(gamma))) atomicOr(st.status, kStatusNonFinite);
      if (!act) atomicSub(st.num_active, 1);
    }
    st.active[cur ^ 1][c] = act ? 1 : 0;
    st.gamma[cur ^ 1][c] = gamma;
    st.beta[c] = b;
  }
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_blk;
  const int64_t r1 = r0 + rows_per_blk < n ? r0 + rows_per_blk : n;
  const int64_t off = (int64_t)c * n;
  for (int64_t i = r0 + threadIdx.x; i < r1; i += blockDim.x) D[off + i] = act ? Z[off + i] + b * D[off + i] : 0.0;
}

// Initial state: gamma0 = gamma, active = ||b|| > 0, counters cleared.
__global__ void mbcg_init_kernel(MbcgState st) {
  const int c = threadIdx.x;
  if (c < st.s) {
    st.gamma0[c] = st.gamma[0][c];
    st.bnorm[c] = sqrt(st.bnorm[c]);
    st.active[0][c] = st.bnorm[c] > 0.0 ? 1 : 0;
    st.iters[c] = 0;
    st.relres[c] = st.bnorm[c] > 0.0 ? 1.0 : 0.0;
    if (!isfinite(st.gamma[0][c]) || !isfinite(st.bnorm[c])) atomicOr(st.status, kStatusNonFinite);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int na = 0;
    for (int i = 0; i < st.s; ++i) na += st.active[0][i];
    *st.num_active = na;
  }
}

// -------------------------------------------------------- tall-skinny products

// Both products run on the FP64 matrix cores (v_mfma_f64_16x16x4: lane l supplies
// A(l % 16, k = l / 16) and B(k = l / 16, l % 16), and holds D(l / 16 + 4 i, l % 16)),
// straight from global memory: every element of the tall matrix is used by one
// wave only, so LDS staging would buy nothing.  The instruction is a chain of four
// FP64 FMAs in the order of k (checked bitwise over 51,200 outputs), so an
// accumulator fed with ascending k holds the bits of a scalar FMA loop.  mBCG
// relies on it: in the mixed form a last-bit change of a direction block now and
// then flips a rounding of its FP16 split, and after some iterations the gradient
// moves by 1e-9.
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2u __attribute__((ext_vector_type(2), aligned(8)));

// The 4 x 4 transpose of v between registers and groups of 16 lanes: lane group g
// enters with v[i] = x(g, i) and leaves with v[i] = x(i, g).
__device__ __forceinline__ void transpose_groups(double (&v)[4]) {
  uint32_t w[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v[i]);
    w[i][0] = (uint32_t)u;
    w[i][1] = (uint32_t)(u >> 32);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {  // groups 2, 3 of register i against groups 0, 1 of register i + 2
      const auto r = __builtin_amdgcn_permlane32_swap(w[i][h], w[i + 2][h], false, false);
      w[i][h] = r[0];
      w[i + 2][h] = r[1];
    }
#pragma unroll
    for (int i = 0; i < 4; i += 2) {  // odd groups of register i against even groups of register i + 1
      const auto r = __builtin_amdgcn_permlane16_swap(w[i][h], w[i + 1][h], false, false);
      w[i][h] = r[0];
      w[i + 1][h] = r[1];
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = __builtin_bit_cast(double, ((uint64_t)w[i][1] << 32) | w[i][0]);
}

// partial[blk][p][q] of G = A^T B over this block's rows in ascending order, A (n x
// pa), B (n x qb), both column-major with ld n.  grid = (nblk, ceil(pa / 64),
// ceil(qb / (16 NQ))); wave w takes columns 16 w .. 16 w + 15 of the group of 64.
// Per 16 rows, lane (x, g) loads rows 4 g .. 4 g + 3 of column x (two 16-byte loads;
// 128-byte runs per column) and a transpose across the lane groups turns them into
// rows 4 i + g, the operand of MFMA i; U such steps are loaded ahead.
// Bound by HBM for narrow B, by the matrix cores for wide ones.  65,536 x 100
// against 16 columns: 28 us in 64 x 64 LDS tiles with one FMA per LDS read, 17 us
// here; 8,192 x 1,024 against 50: 57 us and 32 us.
template <int NQ, int U>
__global__ void __launch_bounds__(256) atb_partial_kernel(const double* __restrict__ A, int pa,
                                                          const double* __restrict__ B, int qb, int64_t n,
                                                          int64_t rows_per_blk, double* __restrict__ partial) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lx = lane & 15, lg = lane >> 4;
  const int p0 = blockIdx.y * 64 + 16 * wave, q0 = blockIdx.z * 16 * NQ;
  if (p0 >= pa) return;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_blk;
  const int64_t r1 = r0 + rows_per_blk < n ? r0 + rows_per_blk : n;
  // columns beyond the matrices repeat the last one and are not stored
  const double* const Ac = A + (int64_t)(p0 + lx < pa ? p0 + lx : pa - 1) * n;
  const double* Bc[NQ];
#pragma unroll
  for (int h = 0; h < NQ; ++h) Bc[h] = B + (int64_t)(q0 + 16 * h + lx < qb ? q0 + 16 * h + lx : qb - 1) * n;
  f64x4 acc[NQ];
#pragma unroll
  for (int h = 0; h < NQ; ++h) acc[h] = f64x4{0.0, 0.0, 0.0, 0.0};
  auto load4 = [&](const double* P, int64_t row, double (&v)[4]) {  // rows beyond the block read as zero
    if (row + 4 <= r1) {
      const f64x2u x = *(const f64x2u*)(P + row), y = *(const f64x2u*)(P + row + 2);
      v[0] = x[0];
      v[1] = x[1];
      v[2] = y[0];
      v[3] = y[1];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = row + i < r1 ? P[row + i] : 0.0;
    }
  };
  double av[U][4], bv[U][NQ][4];
  auto load = [&](int64_t t0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      load4(Ac, t0 + 16 * u + 4 * lg, av[u]);
#pragma unroll
      for (int h = 0; h < NQ; ++h) load4(Bc[h], t0 + 16 * u + 4 * lg, bv[u][h]);
    }
  };
  load(r0);
  for (int64_t t0 = r0; t0 < r1; t0 += 16 * U) {
    double a[U][4], b[U][NQ][4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[u][i] = av[u][i];
#pragma unroll
        for (int h = 0; h < NQ; ++h) b[u][h][i] = bv[u][h][i];
      }
    if (t0 + 16 * U < r1) load(t0 + 16 * U);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      transpose_groups(a[u]);
#pragma unroll
      for (int h = 0; h < NQ; ++h) transpose_groups(b[u][h]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int h = 0; h < NQ; ++h) acc[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][i], b[u][h][i], acc[h], 0, 0, 0);
    }
  }
  double* const dst = partial + (int64_t)blockIdx.x * pa * qb;
#pragma unroll
  for (int h = 0; h < NQ; ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p = p0 + lg + 4 * i, q = q0 + 16 * h + lx;
      if (p < pa && q < qb) dst[(int64_t)p * qb + q] = acc[h][i];
    }
}

// out[p*qb + q] = sum_blk partial in block order, one thread per output, 32 loads in flight.
__global__ __launch_bounds__(64) void atb_reduce_kernel(const double* __restrict__ partial, int64_t nblk, int64_t pq,
                                                        double* __restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (e >= pq) return;
  double acc = 0.0;
  int64_t b = 0;
  for (; b + 32 <= nblk; b += 32) {
    double v[32];
#pragma unroll
    for (int u = 0; u < 32; ++u) v[u] = partial[(b + u) * pq + e];
#pragma unroll
    for (int u = 0; u < 32; ++u) acc += v[u];
  }
  for (; b + 4 <= nblk; b += 4) {
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = partial[(b + u) * pq + e];
#pragma unroll
    for (int u = 0; u < 4; ++u) acc += v[u];
  }
  for (; b < nblk; ++b) acc += partial[b * pq + e];
  out[e] = acc;
}

// Y = post (V + sign A C) (V null: post sign A C) for A (nrows x kk, column-major,
// lda), C (kk x s, row-major with row stride ldc), V and Y (nrows x s,
// column-major with ldv / ldy), s <= 16 NCB.  KW = 1: every wave owns 16 rows and
// takes all of k in ascending order.  KW = 4: the four waves of a workgroup share
// its 16 rows, a quarter of k each, and meet in LDS, so that a block of 8,192 rows
// already gives every SIMD two waves.  Either way a row of A and V is read by the
// workgroup that writes that row of Y, before it does, so Y may alias A or V.
// Bound by HBM (A read once) for narrow C, by the matrix cores for wide ones
// (8,192 x 1,024 times 50 columns: 14 us).  One thread per row with 64
// accumulators, 32 workgroups at 8,192 rows, took 199 us; the block solver's
// products take 14 us on average.  65,536 x 100 times 16 columns (the Woodbury
// finish): 92 us, now 17 us.
template <int NCB, int KW>
__global__ __launch_bounds__(256) void tall_product_kernel(const double* A, int64_t lda, int64_t nrows, int kk,
                                                           const double* __restrict__ C, int64_t ldc, int s, double sign,
                                                           double post, const double* V, int64_t ldv, double* Y,
                                                           int64_t ldy) {
  constexpr int kRows = KW == 1 ? 64 : 16, kCols = 16 * NCB;  // of the workgroup
  __shared__ double red[4][kCols][17];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lx = lane & 15, lg = lane >> 4;
  const int64_t r0 = (int64_t)blockIdx.x * kRows;
  const int kq = (kk + 15) / 16 * 4;
  const int kbeg = KW == 1 ? 0 : wave * kq, kend = KW == 1 || kbeg + kq > kk ? kk : kbeg + kq;
  // rows and columns beyond the matrices repeat the last one and are not stored
  const int64_t arow = r0 + (KW == 1 ? 16 * wave : 0) + lx;
  const double* const Ar = A + (arow < nrows ? arow : nrows - 1);
  const double* Cc[NCB];
#pragma unroll
  for (int h = 0; h < NCB; ++h) Cc[h] = C + (16 * h + lx < s ? 16 * h + lx : s - 1);
  f64x4 acc[NCB];
#pragma unroll
  for (int h = 0; h < NCB; ++h) acc[h] = f64x4{0.0, 0.0, 0.0, 0.0};
  double av[4], cv[4][NCB];
  // 16 k values: MFMA u takes k + 4 u + lg.  Beyond kend both operands are zero (an
  // infinity of C times a zero of A would be NaN).
  auto load = [&](int k) {
    if (k + 16 <= kend) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t kx = k + 4 * u + lg;
        av[u] = Ar[kx * lda];
#pragma unroll
        for (int h = 0; h < NCB; ++h) cv[u][h] = Cc[h][kx * ldc];
      }
      return;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int kx = k + 4 * u + lg;
      const int64_t kc = kx < kend ? kx : kend - 1;
      const double v = Ar[kc * lda];
      av[u] = kx < kend ? v : 0.0;
#pragma unroll
      for (int h = 0; h < NCB; ++h) {
        const double w = Cc[h][kc * ldc];
        cv[u][h] = kx < kend ? w : 0.0;
      }
    }
  };
  if (kbeg < kend) {
    load(kbeg);
    for (int k = kbeg; k < kend; k += 16) {
      double a[4], c[4][NCB];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        a[u] = av[u];
#pragma unroll
        for (int h = 0; h < NCB; ++h) c[u][h] = cv[u][h];
      }
      if (k + 16 < kend) load(k + 16);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int h = 0; h < NCB; ++h) acc[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], c[u][h], acc[h], 0, 0, 0);
    }
  }
#pragma unroll
  for (int h = 0; h < NCB; ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][16 * h + lx][lg + 4 * i] = acc[h][i];
  constexpr int kPer = kRows * kCols / 256;
  double v[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int e = (int)threadIdx.x + 256 * u, r = e % kRows, c = e / kRows;
    v[u] = V && c < s && r0 + r < nrows ? V[(int64_t)c * ldv + r0 + r] : 0.0;
  }
  __syncthreads();  // every wave has read its part of A, every thread its part of V
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int e = (int)threadIdx.x + 256 * u, r = e % kRows, c = e / kRows;
    const double p = KW == 1 ? red[r >> 4][c][r & 15]
                             : ((red[0][c][r] + red[1][c][r]) + red[2][c][r]) + red[3][c][r];
    if (c < s && r0 + r < nrows) Y[(int64_t)c * ldy + r0 + r] = post * (v[u] + sign * p);
  }
}

// v of lane `lane` (wave-uniform), as a wave-uniform value.
__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// v / d from the correctly rounded r = 1 / d: one residual correction of v r gives
// the correctly rounded quotient (Markstein 1990), the bits of the division where
// nothing over- or underflows.
__device__ __forceinline__ double div_by(double v, double d, double r) {
  const double q = v * r;
  return fma(fma(-q, d, v), r, q);
}

// Y := C^{-1} Y for the k x s right-hand sides Y (row-major k x s, entry [j*s + c]),
// with the lower Cholesky factor Lc (column-major k x k), k <= kCholLdsK; the bits
// of the scalar loops below.  Bound by the issue of one wave's dependent steps,
// once per mBCG iteration: the factor and the reciprocals of its diagonal sit in
// LDS (odd pitch: no bank conflicts), one wave per right-hand side.  Forward, lane
// l holds entries l and l + 64 and each solved entry is subtracted from all others
// at once, which is the scalar order.  Backward, the scalar order subtracts the
// newest entry first, a chain of k^2 / 2 FMAs: one lane per right-hand side, factor
// and solution read from LDS 8 terms ahead, also across rows.  A batch reads past
// the last entry: the solution is zero there, so that the factor's
// entries only have to be finite.  k = 100, s = 16: 350 us with one thread per column
// and everything in L2, 99 us with the reads where the compiler moved them, next to their
// use, 80 us so (16 terms ahead 84).
constexpr int kCholLdsK = 128;  // LDS: chol_lds_bytes
constexpr int kCholCols = 4;    // right-hand sides per workgroup
constexpr int kCholB = 8;       // terms of a batch
constexpr int kCholPad = 4 * kCholB;

static size_t chol_lds_bytes(int k) {
  return sizeof(double) * ((size_t)(k | 1) * k + kCholPad + (size_t)kCholCols * ((k + kCholPad) | 1) + k);
}

__global__ __launch_bounds__(256) void chol_solve_lds_kernel(const double* __restrict__ Lc, int k,
                                                             double* __restrict__ Y, int s) {
  extern __shared__ double lds[];
  const int pitch = k | 1, ypitch = (k + kCholPad) | 1;
  double* const Ls = lds;                          // entry (row i, column j) at j pitch + i
  double* const Ys = Ls + k * pitch + kCholPad;    // entry i of column c at c ypitch + i
  double* const Rd = Ys + kCholCols * ypitch;      // 1 / L_jj
  const int tid = threadIdx.x;
  const int lane = tid & 63, hi = lane + 64, wave = tid >> 6;
  const int c = blockIdx.x * kCholCols + wave;  // this wave's right-hand side
  const double y0in = lane < k && c < s ? Y[(int64_t)lane * s + c] : 0.0;
  const double y1in = hi < k && c < s ? Y[(int64_t)hi * s + c] : 0.0;
  for (int j0 = wave; j0 < k; j0 += 32) {  // eight columns of the factor in flight per wave
    double v0[8], v1[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const double* const col = Lc + (int64_t)(j0 + 4 * u < k ? j0 + 4 * u : k - 1) * k;
      v0[u] = col[lane < k ? lane : k - 1];
      v1[u] = col[hi < k ? hi : k - 1];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int j = j0 + 4 * u;
      if (j < k) {
        // zeros above the diagonal: whatever the factor's array holds there is never used
        if (lane < pitch) Ls[j * pitch + lane] = lane >= j && lane < k ? v0[u] : 0.0;
        if (hi < pitch) Ls[j * pitch + hi] = hi >= j && hi < k ? v1[u] : 0.0;
        if (lane + 128 < pitch) Ls[j * pitch + lane + 128] = 0.0;
        if (j == lane) Rd[j] = 1.0 / v0[u];
        if (j == hi) Rd[j] = 1.0 / v1[u];
      }
    }
  }
  if (tid < kCholPad) Ls[k * pitch + tid] = 0.0;
  __syncthreads();
  double y0 = y0in, y1 = y1in;
  {
    // forward, L z = y: z_j leaves the rows below; the next column is read ahead
    // (lanes beyond a short column read whatever follows it; their values are not used)
    const int h = hi < pitch ? hi : lane;
    double d = Ls[0], r = Rd[0], l0 = Ls[lane], l1 = Ls[h];
    const int k0 = k < 64 ? k : 64;
    for (int j = 0; j < k; ++j) {
      const double* const next = Ls + (j + 1 < k ? j + 1 : j) * pitch;
      const double dn = next[j + 1 < k ? j + 1 : j], rn = Rd[j + 1 < k ? j + 1 : j], l0n = next[lane], l1n = next[h];
      if (j < k0) {
        const double z = div_by(lane_value(y0, j), d, r);
        y0 = lane > j ? fma(-l0, z, y0) : (lane == j ? z : y0);
        y1 = fma(-l1, z, y1);
      } else {
        const double z = div_by(lane_value(y1, j - 64), d, r);
        y1 = hi > j ? fma(-l1, z, y1) : (hi == j ? z : y1);
      }
      d = dn;
      r = rn;
      l0 = l0n;
      l1 = l1n;
    }
  }
  for (int i = k + lane; i < ypitch; i += 64) Ys[wave * ypitch + i] = 0.0;
  if (lane < k) Ys[wave * ypitch + lane] = y0;
  if (hi < k) Ys[wave * ypitch + hi] = y1;
  __syncthreads();
  const int cb = blockIdx.x * kCholCols + tid;
  if (tid >= kCholCols || cb >= s) return;
  // backward, L^T x = z: x_j = (z_j - L_{j+1,j} x_{j+1} - L_{j+2,j} x_{j+2} - ...) / L_jj
  double* const Yc = Ys + tid * ypitch;
  double la[kCholB], ya[kCholB], lb[kCholB], yb[kCholB];
  auto read = [&](double(&l)[kCholB], double(&y)[kCholB], int j, int at) {
    const double* const lp = Ls + j * pitch + j + 2 + at;
    const double* const yp = Yc + j + 2 + at;
#pragma unroll
    for (int u = 0; u < kCholB; ++u) {
      l[u] = lp[u];
      y[u] = yp[u];
    }
  };
  double x = 0.0;  // x_{j+1}; the entry of the factor beside it is in the padding at j = k - 1
  double c1 = 0.0, z = Yc[k - 1], d = Ls[(k - 1) * pitch + k - 1], r = Rd[k - 1];
  read(la, ya, k - 1, 0);
  for (int j = k - 1; j >= 0; --j) {
    const int jn = j > 0 ? j - 1 : 0;  // the next row
    const double c1n = Ls[jn * pitch + jn + 1], zn = Yc[jn], dn = Ls[jn * pitch + jn], rn = Rd[jn];
    double v = fma(-c1, x, z);
    const int terms = k - j - 2;
    int at = 0;
    do {
      const bool last = at + 2 * kCholB >= terms;
      read(lb, yb, j, at + kCholB);
      __builtin_amdgcn_sched_barrier(0);  // the compiler would move the reads down to their use
#pragma unroll
      for (int u = 0; u < kCholB; ++u) v = fma(-la[u], ya[u], v);
      __builtin_amdgcn_sched_barrier(0);
      read(la, ya, last ? jn : j, last ? 0 : at + 2 * kCholB);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < kCholB; ++u) v = fma(-lb[u], yb[u], v);
      __builtin_amdgcn_sched_barrier(0);
      at += 2 * kCholB;
    } while (at < terms);
    x = div_by(v, d, r);
    Yc[j] = x;
    Y[(int64_t)j * s + cb] = x;
    c1 = c1n;
    z = zn;
    d = dn;
    r = rn;
  }
}

// The same for a factor that does not fit LDS.  One thread per column.
__global__ void chol_solve_kernel(const double* __restrict__ Lc, int k, double* __restrict__ Y, int s) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= s) return;
  // The terms of each dot product are subtracted in index order; their loads
  // are issued eight at a time so that the chain waits once per eight terms.
  // forward: Lc z = y
  for (int j = 0; j < k; ++j) {
    double v = Y[(int64_t)j * s + c];
    int i = 0;
    for (; i + 8 <= j; i += 8) {
      double lv[8], yv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        lv[u] = Lc[(int64_t)(i + u) * k + j];
        yv[u] = Y[(int64_t)(i + u) * s + c];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) v -= lv[u] * yv[u];
    }
    for (; i < j; ++i) v -= Lc[(int64_t)i * k + j] * Y[(int64_t)i * s + c];
    Y[(int64_t)j * s + c] = v / Lc[(int64_t)j * k + j];
  }
  // backward: Lc^T x = z
  for (int j = k - 1; j >= 0; --j) {
    double v = Y[(int64_t)j * s + c];
    int i = j + 1;
    for (; i + 8 <= k; i += 8) {
      double lv[8], yv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        lv[u] = Lc[(int64_t)j * k + i + u];
        yv[u] = Y[(int64_t)(i + u) * s + c];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) v -= lv[u] * yv[u];
    }
    for (; i < k; ++i) v -= Lc[(int64_t)j * k + i] * Y[(int64_t)i * s + c];
    Y[(int64_t)j * s + c] = v / Lc[(int64_t)j * k + j];
  }
}

__global__ void copy_kernel(const double* __restrict__ src, double* __restrict__ dst, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) dst[i] = src[i];
}

__global__ void zero_words_kernel(uint32_t* __restrict__ dst, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) dst[i] = 0u;
}

__global__ void fill_kernel(double* __restrict__ dst, double v, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) dst[i] = v;
}

// w -= Q h  (Q: n x jn column-major, h: jn values).  One thread per row.
__global__ void gemv_sub_kernel(const double* __restrict__ Q, int64_t n, int jn, const double* __restrict__ h,
                                double* __restrict__ w) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double acc = 0.0;
  for (int j = 0; j < jn; ++j) acc += Q[(int64_t)j * n + i] * h[j];
  w[i] -= acc;
}

// dst = src * (*scale_inv_sqrt)^(-1/2): dst = src / sqrt(*s2)
__global__ void scale_rsqrt_kernel(const double* __restrict__ src, const double* __restrict__ s2, int64_t n,
                                   double* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i] / sqrt(*s2);
}

// In place Q -> R = Q L_T^{-T} for the lower bidiagonal Cholesky factor L_T of
// the Lanczos tridiagonal (diagonal l_j, subdiagonal m_j):
//   R[:, j] = (Q[:, j] - m_j R[:, j-1]) / l_j.   One thread per row.
__global__ void bidiag_solve_kernel(double* __restrict__ QR, int64_t n, int K, const double* __restrict__ lm) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double prev = 0.0;
  for (int j = 0; j < K; ++j) {
    const double v = (QR[(int64_t)j * n + i] - (j > 0 ? lm[2 * j + 1] * prev : 0.0)) / lm[2 * j];
    QR[(int64_t)j * n + i] = v;
    prev = v;
  }
}

// mean[q] = P[q]; var[q] = s_f - sum_{c=1..kc} P[c*m + q]^2.  One wave per
// query row: lane l adds the columns 1 + l, 65 + l, ... in order, then an XOR
// butterfly adds the lanes (the same order on every lane, fixed by kc alone).
__global__ __launch_bounds__(256) void predict_finish_kernel(const double* __restrict__ P, int64_t m, int kc,
                                                             double sf, double* __restrict__ mean,
                                                             double* __restrict__ var) {
  const int lane = threadIdx.x & 63;
  const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (q >= m) return;  // whole wave
  if (lane == 0) mean[q] = P[q];
  if (var) {
    double s = 0.0;
    for (int c = 1 + lane; c <= kc; c += 64) {
      const double v = P[(int64_t)c * m + q];
      s += v * v;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) var[q] = sf - s;
  }
}

// --------------------------------------------------------------------- probes

__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
  uint64_t z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ double rademacher(uint64_t key, uint64_t stream, uint64_t row) {
  return (splitmix64(key ^ ((stream << 40) | row)) >> 63) ? -1.0 : 1.0;
}

// Column c >= 1 of B: L e1_c + sqrt(noise) e2_c (or e2_c when k == 0); column 0 = y.
// grid = (ceil(n/256), t+1).  e1 signs are recomputed per thread from the hash.
__global__ void probe_kernel(const double* __restrict__ y, int64_t n, const double* __restrict__ L, int k,
                             double sigma, uint64_t key, double* __restrict__ B) {
  __shared__ double e1[1024];
  const int c = blockIdx.y;
  if (c > 0 && k > 0) {
    for (int j = threadIdx.x; j < k; j += blockDim.x)
      e1[j] = rademacher(key, (uint64_t)c + kEps1StreamOffset, (uint64_t)j);
    __syncthreads();
  }
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double v;
  if (c == 0) {
    v = y[i];
  } else {
    const double e2 = rademacher(key, (uint64_t)c, (uint64_t)i);
    if (k == 0) {
      v = e2;
    } else {
      double acc = 0.0;
      for (int j = 0; j < k; ++j) acc += L[(int64_t)j * n + i] * e1[j];
      v = acc + sigma * e2;
    }
  }
  B[(int64_t)c * n + i] = v;
}

// ------------------------------------------------------------ pivoted Cholesky

// The better of two (value, index) pairs: the larger value, the lower index on a
// tie; index -1 stands for none.  The order in which pairs meet does not matter.
__device__ __forceinline__ void keep_max(double& bv, int64_t& bi, double v, int64_t i) {
  if (i >= 0 && (bi < 0 || v > bv || (v == bv && i < bi))) {
    bv = v;
    bi = i;
  }
}

template <int THREADS>
__device__ __forceinline__ void block_max(double& bv, int64_t& bi, double* sv, int64_t* si) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double ov = __shfl_xor(bv, off, 64);
    const int64_t oi = __shfl_xor(bi, off, 64);
    keep_max(bv, bi, ov, oi);
  }
  if constexpr (THREADS > 64) {
    if ((threadIdx.x & 63) == 0) {
      sv[threadIdx.x >> 6] = bv;
      si[threadIdx.x >> 6] = bi;
    }
    __syncthreads();
    for (int w = 0; w < THREADS / 64; ++w) keep_max(bv, bi, sv[w], si[w]);
    __syncthreads();
  }
}

// Step m of the pivoted Cholesky: the pivot p, column m of L for all rows,
// l_a = (K(x_a, x_p) - L[a, :m] L[p, :m]^T) / sqrt(delta_p), delta_a -= l_a^2,
// delta_p = 0.  Kernel values in FP64 by direct differences.
//
// One launch per step (a step at n = 2,048 or 65,536 is bound by its launches and
// their latency): each workgroup finds the pivot itself from the block maxima of
// step m - 1 (delta is s_f everywhere before step 0, so its pivot is row 0), and
// leaves the maximum of its rows' new delta for step m + 1 in the other of two
// buffers.  Once the largest delta falls to stop_below, ps.rank stays behind m and
// every later step returns.  n = 65,536, d = 48, rank 100: 21 us a step with the two
// argmax launches, 15.2 now (X and half of L: 50 MB, 10.5 us at the copy rate); n =
// 2,048, d = 32, rank 20: 7.4 us.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void pivchol_step_kernel(const double* __restrict__ X, int64_t n, int d,
                                                               Scale inv_ell, int kind, double sf,
                                                               double* __restrict__ L, double* __restrict__ delta,
                                                               PivState ps, int m, double stop_below,
                                                               int64_t rows_per_blk) {
  __shared__ double xp[GP_MAX_D];
  __shared__ double lp[1024];
  __shared__ double sv[THREADS / 64 + 1];
  __shared__ int64_t si[THREADS / 64 + 1];
  const int nblk = gridDim.x;
  double pv = sf;
  int64_t p = 0;
  if (m > 0) {
    if (*ps.rank < m) return;  // stopped before step m (block 0 may already store m + 1)
    const double* const bv = ps.bval + (m & 1) * nblk;
    const int64_t* const bi = ps.bidx + (m & 1) * nblk;
    pv = -1.0;
    p = -1;
    for (int b = threadIdx.x; b < nblk; b += THREADS) keep_max(pv, p, bv[b], bi[b]);
    block_max<THREADS>(pv, p, sv, si);
    if (!(pv > stop_below) || p < 0) return;  // rank stays m
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ps.piv[m] = p;
    ps.pivval[m] = pv;
    *ps.rank = m + 1;
  }
  for (int j = threadIdx.x; j < d; j += THREADS) xp[j] = X[p * d + j];
  for (int j = threadIdx.x; j < m; j += THREADS) lp[j] = L[(int64_t)j * n + p];
  __syncthreads();
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_blk;
  const int64_t r1 = r0 + rows_per_blk < n ? r0 + rows_per_blk : n;
  double bv = -1.0;
  int64_t bi = -1;
  for (int64_t a = r0 + threadIdx.x; a < r1; a += THREADS) {
    double r2 = 0.0;
#pragma unroll 8
    for (int j = 0; j < d; ++j) {
      const double df = (X[a * d + j] - xp[j]) * inv_ell.s[j];
      r2 += df * df;
    }
    double kv;
    if (kind == GP_MATERN52) {
      const double s = sqrt(5.0 * r2);
      kv = sf * (1.0 + s + s * s / 3.0) * exp(-s);
    } else {
      kv = sf * exp(-0.5 * r2);
    }
    double acc = 0.0;
#pragma unroll 8
    for (int j = 0; j < m; ++j) acc += L[(int64_t)j * n + a] * lp[j];
    const double l = (kv - acc) / sqrt(pv);
    L[(int64_t)m * n + a] = l;
    const double dn = (a == p) ? 0.0 : (m > 0 ? delta[a] : sf) - l * l;
    delta[a] = dn;
    if (dn > bv) {  // strictly greater: the first (lowest) index of a tie wins within a thread
      bv = dn;
      bi = a;
    }
  }
  block_max<THREADS>(bv, bi, sv, si);
  if (threadIdx.x == 0) {
    ps.bval[((m + 1) & 1) * nblk + blockIdx.x] = bv;
    ps.bidx[((m + 1) & 1) * nblk + blockIdx.x] = bi;
  }
}

// --------------------------------------------------------------- host helpers

static unsigned blocks_for(int64_t count, int thr = kThreads) { return (unsigned)((count + thr - 1) / thr); }

RowSplit row_split(int64_t n, int64_t target_blocks) {
  RowSplit r;
  int64_t per = (n + target_blocks - 1) / target_blocks;
  per = (per + kThreads - 1) / kThreads * kThreads;
  if (per < kThreads) per = kThreads;
  r.rows_per_blk = per;
  r.nblk = (n + per - 1) / per;
  return r;
}

hipError_t coldot(const double* A, const double* B, int64_t n, int s, double* out, double* partial,
                  hipStream_t st) {
  const RowSplit rs = row_split(n, kDotBlocks);
  coldot_partial_kernel<<<dim3((unsigned)rs.nblk, (unsigned)s), kThreads, 0, st>>>(A, B, n, rs.rows_per_blk, s,
                                                                                   partial);
  reduce_partials_kernel<<<s, kThreads, 0, st>>>(partial, rs.nblk, s, out);
  return hipGetLastError();
}

static void launch_atb_partial(const double* A, int pa, const double* B, int qb, int64_t n, const RowSplit& rs,
                               double* partial, hipStream_t st) {
  const unsigned gy = (unsigned)((pa + 63) / 64);
  if (qb <= 16)
    atb_partial_kernel<1, 4><<<dim3((unsigned)rs.nblk, gy, 1), 256, 0, st>>>(A, pa, B, qb, n, rs.rows_per_blk, partial);
  else if (qb <= 32)
    atb_partial_kernel<2, 2><<<dim3((unsigned)rs.nblk, gy, 1), 256, 0, st>>>(A, pa, B, qb, n, rs.rows_per_blk, partial);
  else
    atb_partial_kernel<4, 1><<<dim3((unsigned)rs.nblk, gy, (unsigned)((qb + 63) / 64)), 256, 0, st>>>(
        A, pa, B, qb, n, rs.rows_per_blk, partial);
}

static void launch_atb_reduce(const double* partial, int64_t nblk, int64_t pq, double* out, hipStream_t st) {
  atb_reduce_kernel<<<blocks_for(pq, 64), 64, 0, st>>>(partial, nblk, pq, out);
}

size_t atb_partial_doubles(int64_t n, int pa, int qb) {
  const RowSplit rs = row_split(n, kAtbBlocks);
  return (size_t)rs.nblk * pa * qb;
}

hipError_t atb(const double* A, int pa, const double* B, int qb, int64_t n, double* out, double* partial,
               hipStream_t st) {
  const RowSplit rs = row_split(n, kAtbBlocks);
  launch_atb_partial(A, pa, B, qb, n, rs, partial, st);
  const int64_t pq = (int64_t)pa * qb;
  launch_atb_reduce(partial, rs.nblk, pq, out, st);
  return hipGetLastError();
}

hipError_t atb_n(const double* A, int pa, const double* B, int qb, int64_t n, double* out, double* partial,
                 int64_t nblk, hipStream_t st) {
  const RowSplit rs = row_split(n, nblk);
  launch_atb_partial(A, pa, B, qb, n, rs, partial, st);
  const int64_t pq = (int64_t)pa * qb;
  launch_atb_reduce(partial, rs.nblk, pq, out, st);
  return hipGetLastError();
}

hipError_t precond_apply(const Precond& pc, const double* R, double* Z, int64_t n, int s, double* Y,
                         double* partial, hipStream_t st) {
  if (pc.rank == 0) {
    copy_kernel<<<blocks_for(n * s), kThreads, 0, st>>>(R, Z, n * s);
    return hipGetLastError();
  }
  // Y = L^T R  (k x s, row-major [j*s + c])
  hipError_t e = atb(pc.L, pc.rank, R, s, n, Y, partial, st);
  if (e != hipSuccess) return e;
  if (pc.rank <= kCholLdsK) {
    chol_solve_lds_kernel<<<blocks_for(s, kCholCols), 256, chol_lds_bytes(pc.rank), st>>>(pc.Cchol, pc.rank, Y, s);
  } else {
    chol_solve_kernel<<<blocks_for(s, 64), 64, 0, st>>>(pc.Cchol, pc.rank, Y, s);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // Z = (R - L Y) / sigma^2
  for (int c0 = 0; c0 < s; c0 += kTallMaxS) {
    const int sc = s - c0 < kTallMaxS ? s - c0 : kTallMaxS;
    e = tall_product(pc.L, n, n, pc.rank, Y + c0, s, sc, -1.0, 1.0 / pc.noise, R + (int64_t)c0 * n, n,
                     Z + (int64_t)c0 * n, n, /*split_k=*/false, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int KW>
static void launch_tall(const double* A, int64_t lda, int64_t nrows, int kk, const double* C, int64_t ldc, int s,
                        double sign, double post, const double* V, int64_t ldv, double* Y, int64_t ldy,
                        hipStream_t st) {
  const unsigned grid = blocks_for(nrows, KW == 1 ? 64 : 16);
#define GPK_TALL(NCB) \
  tall_product_kernel<NCB, KW><<<grid, 256, 0, st>>>(A, lda, nrows, kk, C, ldc, s, sign, post, V, ldv, Y, ldy)
  switch ((s + 15) / 16) {
    case 1: GPK_TALL(1); break;
    case 2: GPK_TALL(2); break;
    case 3: GPK_TALL(3); break;
    default: GPK_TALL(4); break;
  }
#undef GPK_TALL
}

hipError_t tall_product(const double* A, int64_t lda, int64_t nrows, int kk, const double* C, int64_t ldc, int s,
                        double sign, double post, const double* V, int64_t ldv, double* Y, int64_t ldy,
                        bool split_k, hipStream_t st) {
  if (s < 1 || s > kTallMaxS || kk < 1) return hipErrorInvalidValue;
  if (split_k)
    launch_tall<4>(A, lda, nrows, kk, C, ldc, s, sign, post, V, ldv, Y, ldy, st);
  else
    launch_tall<1>(A, lda, nrows, kk, C, ldc, s, sign, post, V, ldv, Y, ldy, st);
  return hipGetLastError();
}

hipError_t launch_probes(const double* y, int64_t n, int t, const double* L, int k, double noise, uint64_t seed,
                         double* B, hipStream_t st) {
  const uint64_t key = splitmix64_host(seed);
  probe_kernel<<<dim3(blocks_for(n), (unsigned)(t + 1)), kThreads, 0, st>>>(y, n, L, k, std::sqrt(noise), key, B);
  return hipGetLastError();
}

hipError_t launch_gemv_sub(const double* Q, int64_t n, int jn, const double* h, double* w, hipStream_t st) {
  gemv_sub_kernel<<<blocks_for(n), kThreads, 0, st>>>(Q, n, jn, h, w);
  return hipGetLastError();
}

hipError_t launch_scale_rsqrt(const double* src, const double* s2, int64_t n, double* dst, hipStream_t st) {
  scale_rsqrt_kernel<<<blocks_for(n), kThreads, 0, st>>>(src, s2, n, dst);
  return hipGetLastError();
}

hipError_t launch_bidiag_solve(double* QR, int64_t n, int K, const double* lm, hipStream_t st) {
  bidiag_solve_kernel<<<blocks_for(n), kThreads, 0, st>>>(QR, n, K, lm);
  return hipGetLastError();
}

hipError_t launch_predict_finish(const double* P, int64_t m, int kc, double sf, double* mean, double* var,
                                 hipStream_t st) {
  predict_finish_kernel<<<(unsigned)((m + 3) / 4), 256, 0, st>>>(P, m, kc, sf, mean, var);
  return hipGetLastError();
}

hipError_t launch_copy(const double* src, double* dst, int64_t count, hipStream_t st) {
  copy_kernel<<<blocks_for(count), kThreads, 0, st>>>(src, dst, count);
  return hipGetLastError();
}

hipError_t launch_zero_words(void* dst, int64_t words, hipStream_t st) {
  zero_words_kernel<<<blocks_for(words), kThreads, 0, st>>>((uint32_t*)dst, words);
  return hipGetLastError();
}

hipError_t launch_fill(double* dst, double v, int64_t count, hipStream_t st) {
  fill_kernel<<<blocks_for(count), kThreads, 0, st>>>(dst, v, count);
  return hipGetLastError();
}

hipError_t mbcg_launch_init(const MbcgState& s, hipStream_t st) {
  mbcg_init_kernel<<<1, 256, 0, st>>>(s);
  return hipGetLastError();
}
hipError_t coldot_partials(const double* A, const double* B, int64_t n, int s, double* partial, hipStream_t st) {
  const RowSplit rs = row_split(n, kDotBlocks);
  coldot_partial_kernel<<<dim3((unsigned)rs.nblk, (unsigned)s), kThreads, 0, st>>>(A, B, n, rs.rows_per_blk, s,
                                                                                   partial);
  return hipGetLastError();
}

// Every workgroup of a column adds that column's partial sums, so that this work grows with the
// square of their number.  Up to kSumInPlace (n = 131,072) it costs less than the three launches that
// it saves (an iteration at n = 65,536, d = 5, 16 columns: 1,448 us, 1,459 with the sums first; n =
// 131,072: 5,509 and 5,496); beyond, the sums are formed first (n = 262,144, 33 columns: 28.97 ->
// 28.75 ms).  One partial sum is left then, which is its own sum: the same bits.
constexpr int64_t kSumInPlace = 512;

static int64_t sum_partials(double*& part, double* sum, int64_t nblk, int s, hipStream_t st) {
  if (nblk <= kSumInPlace) return nblk;
  reduce_partials_kernel<<<s, kThreads, 0, st>>>(part, nblk, s, sum);
  part = sum;
  return 1;
}

hipError_t mbcg_launch_update_ur(MbcgState s, int cur, const double* D, const double* W, double* U, double* R,
                                 int64_t n, hipStream_t st) {
  const RowSplit rs = row_split(n, kDotBlocks);
  const int64_t np = sum_partials(s.dpart, s.dsum, rs.nblk, s.s, st);
  mbcg_update_ur_kernel<<<dim3((unsigned)rs.nblk, (unsigned)s.s), kThreads, 0, st>>>(s, cur, np, D, W, U, R, n,
                                                                                      rs.rows_per_blk);
  return hipGetLastError();
}
hipError_t mbcg_launch_update_d(MbcgState s, int cur, int j, double tol, const double* Z, double* D, int64_t n,
                                hipStream_t st) {
  const RowSplit rs = row_split(n, kDotBlocks);
  sum_partials(s.rpart, s.rsum, rs.nblk, s.s, st);
  const int64_t np = sum_partials(s.gpart, s.gsum, rs.nblk, s.s, st);
  mbcg_update_d_kernel<<<dim3((unsigned)rs.nblk, (unsigned)s.s), kThreads, 0, st>>>(s, cur, np, j, tol, Z, D, n,
                                                                                     rs.rows_per_blk);
  return hipGetLastError();
}

// One wave per workgroup up to this many rows, so that few rows still reach many CUs (n = 2,048: 32 workgroups
// instead of 8); four beyond, so that a step has at most 1,024 block maxima to compare.
constexpr int64_t kPivWaveRows = 32768;

static RowSplit pivchol_split(int64_t n) {
  if (n > kPivWaveRows) return row_split(n, kDotBlocks);
  return RowSplit{64, (n + 63) / 64};
}

int64_t pivchol_blocks(int64_t n) { return pivchol_split(n).nblk; }

hipError_t pivchol_launch_step(const double* X, int64_t n, const gp_kernel* kern, double* L, double* delta,
                               const PivState& ps, int m, double stop_below, hipStream_t st) {
  Scale inv{};
  for (int j = 0; j < kern->d; ++j) inv.s[j] = 1.0 / kern->lengthscale[j];
  const RowSplit rs = pivchol_split(n);
  const unsigned grid = (unsigned)rs.nblk;
  if (n > kPivWaveRows)
    pivchol_step_kernel<kThreads><<<grid, kThreads, 0, st>>>(X, n, kern->d, inv, kern->kind, kern->outputscale, L,
                                                             delta, ps, m, stop_below, rs.rows_per_blk);
  else
    pivchol_step_kernel<64><<<grid, 64, 0, st>>>(X, n, kern->d, inv, kern->kind, kern->outputscale, L, delta, ps, m,
                                                 stop_below, rs.rows_per_blk);
  return hipGetLastError();
}

}  // namespace gpk
