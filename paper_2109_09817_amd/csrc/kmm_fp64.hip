// The FP64 form of the kernel-matrix products (low-noise regime).
#include "internal.h"

#include <algorithm>
#include <cmath>

namespace gpk {

constexpr int kF64Chunk = 32;  // points per LDS chunk
constexpr int kF64Cols = 64;   // V columns per workgroup
constexpr int kF64Rows = 64;   // output rows per workgroup

// The low-noise regime (sigma^2 down to 1e-8, Sec. 3.2 and Sec. 4) needs K_hat V
// to FP64 accuracy.  Both contractions run on the FP64 matrix cores
// (v_mfma_f64_16x16x4: lane l supplies A(l % 16, k = l / 16) and B(k = l / 16,
// l % 16), and holds D(l / 16 + 4 i, l % 16)).  A workgroup owns 64 output rows,
// up to 64 columns and one split of the b range; wave w owns rows 16 w .. 16 w
// + 15, their scaled features held in registers as the B operand.  Per 32-point
// chunk of the b stream (scaled points, norms and V values staged in LDS), for
// each 16-point half: the MFMA gives x_b . x_a with the point along D's rows, so
// after the profile (the accumulator starts at -(n_a + n_b) / 2) register i of
// every lane holds the entries of points 4 i .. 4 i + 3 of that half, exactly the
// A operand of the M V step that contracts over them.  Each entry is evaluated
// once and never leaves registers; the output tile goes through LDS so that the
// stores are coalesced.  The diagonal entry is exactly s_f (m(0) = 1) and
// sigma^2 V is added exactly.
//
// Bound: the FP64 matrix cores, 64 cycles per MFMA and SIMD (24 for the
// distances of a 16 x 32 tile at d = 48, 8 per 16 columns of V) plus the
// profile's FP64 VALU (30 instructions of 4 cycles per entry), which mostly adds
// to them.  So the profile is branch-free and runs four entries in step, loads
// are clamped instead of predicated one by one, and the b range is split until
// the grid has about kF64Groups workgroups (see f64_split).  One to four columns
// beyond a multiple of 16 (a block of 50 or 17, a single vector) cost four FMAs
// per entry on the VALU instead of a 16-column MFMA block that is mostly padding.
// n = 24,576, t = 50, d = 48: 5.0 ms with predicated loads, one entry at a time
// through sqrt and exp and one or two workgroups per CU; 2.67 ms now (33 TFLOP/s of
// n^2 (d + 2 t)).  Counters there: matrix pipe busy 55% at 2.06 GHz, waves waiting on 19%
// of their cycles, 3.3 LDS conflict cycles per LDS instruction.  Error against a long
// double product on sampled rows 3.0e-15 (5.1e-15 before: one long sum per row).
typedef double f64x4 __attribute__((ext_vector_type(4)));

// m(r) for four entries at once from h = -S / 2, S = r^2 scaled as for the mixed
// form (profile_coordinate_scale): u = sqrt(S), m = (1 + u ln2 + (u ln2)^2 / 3) 2^-u
// (RBF: 2^-S).  S is kept above 1e-300, where m is 1 to rounding, and the exponent
// below 1100, where 2^-u is 0.
//   sqrt: the hardware's reciprocal square root (about 2^-23), one coupled Newton
//   step for sqrt and half its reciprocal (Goldschmidt 1964; 2^-46), one residual
//   correction, which leaves the rounding of the last operation.
//   2^-u: -u = k + f, f in [-1/2, 1/2] (exact), and the degree-11 interpolant of 2^f
//   at the Chebyshev nodes (relative error 1e-17).
// Four chains run in step: a single chain waits on every result (FP64 latency is
// twice its issue time), and left to itself the compiler runs the entries one
// after the other to save registers.
#define GPK_STEP4(EXPR)                      \
  _Pragma("unroll") for (int i = 0; i < 4; ++i) { EXPR; } \
  __builtin_amdgcn_sched_barrier(0)

template <int KIND>
__device__ __forceinline__ void profile64x4(const f64x4& h, double (&m)[4]) {
  double x[4], q[4], k[4], p[4];
  GPK_STEP4(x[i] = fmax(-2.0 * h[i], 1e-300));
  if constexpr (KIND == GP_MATERN52) {
    GPK_STEP4(k[i] = __builtin_amdgcn_rsq(x[i]));
    GPK_STEP4(q[i] = x[i] * k[i]);                // g0
    GPK_STEP4(k[i] = 0.5 * k[i]);                 // h0
    GPK_STEP4(p[i] = fma(-q[i], k[i], 0.5));
    GPK_STEP4(q[i] = fma(q[i], p[i], q[i]));
    GPK_STEP4(k[i] = fma(k[i], p[i], k[i]));
    GPK_STEP4(x[i] = fma(-q[i], q[i], x[i]));
    GPK_STEP4(x[i] = fma(x[i], k[i], q[i]));
    GPK_STEP4(x[i] = fmin(x[i], 1100.0));
    GPK_STEP4(q[i] = fma(x[i], M_LN2 * M_LN2 / 3.0, M_LN2));
    GPK_STEP4(q[i] = fma(x[i], q[i], 1.0));
  } else {
    GPK_STEP4(x[i] = fmin(x[i], 1100.0));
  }
  GPK_STEP4(k[i] = __builtin_rint(-x[i]));
  GPK_STEP4(x[i] = -x[i] - k[i]);
  GPK_STEP4(p[i] = fma(4.4558179083360645e-10, x[i], 7.074194297288521e-09));
  GPK_STEP4(p[i] = fma(p[i], x[i], 1.0178057087733941e-07));
  GPK_STEP4(p[i] = fma(p[i], x[i], 1.3215432535912375e-06));
  GPK_STEP4(p[i] = fma(p[i], x[i], 1.5252733841556773e-05));
  GPK_STEP4(p[i] = fma(p[i], x[i], 0.00015403530463724353));
  GPK_STEP4(p[i] = fma(p[i], x[i], 0.001333355814640647));
  GPK_STEP4(p[i] = fma(p[i], x[i], 0.009618129107587256));
  GPK_STEP4(p[i] = fma(p[i], x[i], 0.055504108664821625));
  GPK_STEP4(p[i] = fma(p[i], x[i], 0.24022650695910158));
  GPK_STEP4(p[i] = fma(p[i], x[i], 0.6931471805599453));
  GPK_STEP4(p[i] = fma(p[i], x[i], 1.0));
  GPK_STEP4(m[i] = __builtin_amdgcn_ldexp(p[i], (int)k[i]));
  if constexpr (KIND == GP_MATERN52) {
    GPK_STEP4(m[i] *= q[i]);
  }
}

// Squared scaled norms below this keep S finite; the profile's clamps would turn a NaN
// S into m = 1 and an infinite one into m = 0.  A point at or beyond it (a NaN or
// infinite coordinate, or one some 1e153 lengthscales from the origin) makes every
// product involving it NaN, as in the mixed form never silently wrong.  The preparation
// leaves NaN in the first norm of a block of kF64Block that holds such a point; the
// sweep looks there once, at its end (a test per chunk took up to 4% of it).
constexpr double kF64FarNorm = 0x1p1021;
constexpr int kF64Block = 256;

// sc64[f] = feature scale (thread f < d); nrm[p] = |x_p (.) sc|^2 for p < rows.
__global__ __launch_bounds__(kF64Block) void prep_fp64_kernel(const double* __restrict__ X, int64_t rows, int d, Scale sc,
                                 double* __restrict__ sc64, double* __restrict__ nrm) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p < d) sc64[p] = sc.s[p];
  double s = 0.0;
  if (p < rows) {
    for (int f = 0; f < d; ++f) {
      const double v = X[p * d + f] * sc.s[f];
      s = fma(v, v, s);
    }
  }
  __shared__ int far[kF64Block / 64];
  const int wave_far = __any(!(s < kF64FarNorm));
  if ((threadIdx.x & 63) == 0) far[threadIdx.x >> 6] = wave_far;
  if (threadIdx.x != 0 && p < rows) nrm[p] = s;
  __syncthreads();
  if (threadIdx.x == 0 && p < rows) {
    int any = 0;
#pragma unroll
    for (int w = 0; w < kF64Block / 64; ++w) any |= far[w];
    nrm[p] = any ? __builtin_nan("") : s;
  }
}

struct F64Args {
  const double* Xb;    // n x d points, nb their squared scaled norms
  const double* nb;
  const double* Xa;    // output rows, m x d
  const double* sc;
  const double* V;     // this pass's first column
  double* out;         // likewise
  double* part;        // [split][column][slab row] partial sums, or null: one split, straight to out
  int64_t n, m, ldv, ldo;
  int64_t row0;        // first output row of this slab
  int64_t slab;        // rows of the partial buffer
  int64_t cps;         // chunks per split
  int d, t, square;
  int columns;         // of the whole product
  double sf, noise;
};

// Waves per SIMD asked of the compiler: one form fits four by a register or two and left to itself
// takes one too many (n = 24,576, d = 32, t = 16, RBF: 1.34 ms with three, 1.32 with four).
constexpr int f64_waves(int dp, int kind, int ncb, int rem) {
  return dp == 32 && kind == GP_RBF && ncb == 1 && rem == 0 ? 4 : 2;
}

// Columns c0 .. c0 + live - 1 of the pass, live <= 16 NCB + REM: NCB 16-column blocks
// on the matrix cores, REM columns on the VALU (columns beyond live repeat the
// last one and are not stored).
template <int DP, int KIND, int NCB, int REM>
__global__ __launch_bounds__(256, (f64_waves(DP, KIND, NCB, REM))) void sweep_fp64_kernel(F64Args a, int first_col,
                                                                                          int columns) {
  constexpr int kBLd = DP + 2;           // point rows: a half-wave's operand reads hit distinct banks
  constexpr int kVLd = kF64Chunk + 2;    // V columns, likewise
  constexpr int kOLd = kF64Rows + 1;     // output tile columns
  constexpr int kKs = DP / 4;            // K steps of the distance MFMA
  constexpr int kCols = 16 * NCB + REM;
  constexpr int kVPer = (kCols + 7) / 8;
  constexpr int kStage = kF64Chunk * kBLd + 8 * kVPer * kVLd;
  constexpr int kBuf = kStage > kCols * kOLd ? kStage : kCols * kOLd;
  constexpr int kBPer = kF64Chunk * DP / 256;
  static_assert(kF64Chunk * DP % 256 == 0, "256 threads");
  __shared__ double buf[kBuf];  // the chunk's points [j][f] and V [c][j]; at the end the output tile [c][row]
  __shared__ double Ns[kF64Chunk];
  __shared__ double Sc[DP];
  double* const Bs = buf;
  double* const Vs = buf + kF64Chunk * kBLd;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const int d = a.d;
  const int64_t n = a.n;
  const int64_t a0 = a.row0 + (int64_t)blockIdx.x * kF64Rows;
  const int c0 = first_col + blockIdx.y * kF64Cols;
  const int live = a.t - c0 < columns ? a.t - c0 : columns;
  const int64_t arow = a0 + 16 * wave + lr;          // this lane's row in the products
  const int64_t crow = arow < a.m ? arow : a.m - 1;  // rows beyond m compute row m - 1, not stored
  double xa[kKs];
#pragma unroll
  for (int s = 0; s < kKs; ++s) {
    const int f = 4 * s + lk;
    xa[s] = f < d ? a.Xa[crow * d + f] * a.sc[f] : 0.0;
  }
  double naa = 0.0;
  if (a.square) {
    naa = a.nb[crow];
  } else {  // the sequence of additions of prep_fp64_kernel
    for (int f = 0; f < d; ++f) {
      const double v = a.Xa[crow * d + f] * a.sc[f];
      naa = fma(v, v, naa);
    }
  }
  f64x4 acc[NCB > 0 ? NCB : 1];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) acc[cb] = f64x4{0.0, 0.0, 0.0, 0.0};
  double accr[REM > 0 ? REM : 1];
#pragma unroll
  for (int c = 0; c < REM; ++c) accr[c] = 0.0;
  // Staging: the next chunk's points, V and norms are loaded into registers
  // while the current chunk is computed from LDS.  A chunk's points are 32 d
  // consecutive values; thread tid takes every 256th (offsets clamped into X),
  // and 32 values of every eighth column of V.
  const int nd = kF64Chunk * d;
  int bpos[kBPer];        // LDS position of each point value,
  uint32_t boff[kBPer];   // its byte offset from the chunk's first
  // and its feature's scale, from LDS where the registers would cost a wave per SIMD
  // or spill (t = 16, d = 48: 1.86 ms, 1.98 from registers; t = 50: 2.76, 2.70)
  constexpr bool kRegScale = DP <= 48 && (NCB != 1 || REM > 0);
  double bsc[kRegScale ? kBPer : 1];
  int bf[kRegScale ? 1 : kBPer];
#pragma unroll
  for (int it = 0; it < kBPer; ++it) {
    const int e = tid + 256 * it < nd ? tid + 256 * it : nd - 1;
    bpos[it] = e / d * kBLd + e % d;
    boff[it] = 8u * e;
    if constexpr (kRegScale)
      bsc[it] = a.sc[e % d];
    else
      bf[it] = e % d;
  }
  for (int e = tid; e < kF64Chunk * kBLd; e += 256) Bs[e] = 0.0;  // the features beyond d stay zero
  if (tid < DP) Sc[tid] = tid < d ? a.sc[tid] : 0.0;
  const int vcol = tid >> 5, vj = tid & 31;
  const double* vp[kVPer];  // V of point vj in this thread's columns
#pragma unroll
  for (int it = 0; it < kVPer; ++it)
    vp[it] = a.V + (int64_t)(c0 + (8 * it + vcol < live ? 8 * it + vcol : live - 1)) * a.ldv + vj;
  double bv[kBPer], vv[kVPer], nv;
  // Full chunks add a scalar to offsets and pointers that stay: vector address
  // arithmetic adds to the time of the MFMAs.
  auto load = [&](int64_t c0b) {
    const char* const Xc = (const char*)(a.Xb + c0b * d);
    if (n - c0b >= kF64Chunk) {
#pragma unroll
      for (int it = 0; it < kBPer; ++it) bv[it] = *(const double*)(Xc + boff[it]);
#pragma unroll
      for (int it = 0; it < kVPer; ++it) vv[it] = vp[it][c0b];
      nv = a.nb[c0b + vj];
      return;
    }
    const uint32_t blim = 8u * (uint32_t)((n - c0b) * d - 1);
    const int back = vj >= (int)(n - c0b) ? vj - (int)(n - c0b) + 1 : 0;  // points beyond n repeat the last one
#pragma unroll
    for (int it = 0; it < kBPer; ++it) bv[it] = *(const double*)(Xc + (boff[it] < blim ? boff[it] : blim));
#pragma unroll
    for (int it = 0; it < kVPer; ++it) vv[it] = vp[it][c0b - back];
    nv = a.nb[c0b + vj - back];
  };
  const int64_t b_begin = (int64_t)blockIdx.z * a.cps * kF64Chunk;
  const int64_t b_end = b_begin + a.cps * kF64Chunk < n ? b_begin + a.cps * kF64Chunk : n;
  load(b_begin);
  for (int64_t b0 = b_begin; b0 < b_end; b0 += kF64Chunk) {
    const bool tail = b0 + kF64Chunk > n;
    __syncthreads();  // the previous chunk's readers are done (first: Sc and the zeroed features are written)
    if (tail) {       // points beyond n: their entries are zeroed below, their V here
#pragma unroll
      for (int it = 0; it < kVPer; ++it) vv[it] = b0 + vj < n ? vv[it] : 0.0;
    }
#pragma unroll
    for (int it = 0; it < kBPer; ++it)
      if (tid + 256 * it < nd) Bs[bpos[it]] = bv[it] * (kRegScale ? bsc[kRegScale ? it : 0] : Sc[bf[kRegScale ? 0 : it]]);
#pragma unroll
    for (int it = 0; it < kVPer; ++it) Vs[(8 * it + vcol) * kVLd + vj] = vv[it];
    if (tid < kF64Chunk) Ns[tid] = nv;
    __syncthreads();
    if (b0 + kF64Chunk < b_end) load(b0 + kF64Chunk);
    __builtin_amdgcn_sched_barrier(0);
    // x_b . x_a - (n_a + n_b) / 2 = -r^2 / 2: D(point 16 pb + lk + 4 i, row arow), both halves of the chunk
    f64x4 dt[2];
#pragma unroll
    for (int q = 0; q < 8; ++q) dt[q >> 2][q & 3] = -0.5 * (naa + Ns[16 * (q >> 2) + lk + 4 * (q & 3)]);
#pragma unroll
    for (int s = 0; s < kKs; ++s)
#pragma unroll
      for (int pb = 0; pb < 2; ++pb)
        dt[pb] = __builtin_amdgcn_mfma_f64_16x16x4f64(Bs[(16 * pb + lr) * kBLd + 4 * s + lk], xa[s], dt[pb], 0, 0, 0);
    const bool edge = tail || (a.square && b0 < a0 + kF64Rows && b0 + kF64Chunk > a0);
#pragma unroll
    for (int pb = 0; pb < 2; ++pb) {
      double mt[4];
      profile64x4<KIND>(dt[pb], mt);
      if (edge) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int64_t b = b0 + 16 * pb + lk + 4 * i;
          if (a.square && b == arow) mt[i] = 1.0;
          if (b >= n) mt[i] = 0.0;
        }
      }
      // acc(row, column) += sum over the half's points of M(row, point) V(point, column)
      const double* const Vp = Vs + 16 * pb + lk;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
          acc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(mt[i], Vp[(16 * cb + lr) * kVLd + 4 * i], acc[cb], 0, 0, 0);
#pragma unroll
        for (int c = 0; c < REM; ++c) accr[c] = fma(mt[i], Vp[(16 * NCB + c) * kVLd + 4 * i], accr[c]);
      }
    }
  }
  // acc[cb][i]: row 16 wave + lk + 4 i, column 16 cb + lr -> LDS tile [column][row]
  const double mark = a.nb[kF64Block * lane < n ? kF64Block * lane : 0];  // in flight across the barriers
  __syncthreads();
  double* const Os = buf;
  int* const row_far = (int*)Ns;
  if (lk == 0) row_far[16 * wave + lr] = !(naa < kF64FarNorm);
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
    for (int i = 0; i < 4; ++i) Os[(16 * cb + lr) * kOLd + 16 * wave + lk + 4 * i] = acc[cb][i];
#pragma unroll
  for (int c = 0; c < REM; ++c) {  // row lr's four lanes lk hold every fourth point
    accr[c] += __shfl_xor(accr[c], 16);
    accr[c] += __shfl_xor(accr[c], 32);
    if (lk == 0) Os[(16 * NCB + c) * kOLd + 16 * wave + lr] = accr[c];
  }
  bool far = !(mark < kF64FarNorm);
  for (int64_t p = kF64Block * (64 + lane); p < n; p += 64 * kF64Block) far |= !(a.nb[p] < kF64FarNorm);
  __syncthreads();
  // lane's row (a square product of one point has the exact diagonal only)
  const bool nan = (__any(far) || row_far[lane]) && !(a.square && n == 1);
  auto sum = [&](int c) { return nan ? __builtin_nan("") : Os[c * kOLd + lane]; };
  if (a.part) {
    const int64_t r = (int64_t)blockIdx.x * kF64Rows + lane;
    for (int c = wave; c < live; c += 4) a.part[((int64_t)blockIdx.z * a.t + c0 + c) * a.slab + r] = sum(c);
    return;
  }
  const int64_t ar = a0 + lane;
  if (ar >= a.m) return;
  for (int c = wave; c < live; c += 4) {
    double y = a.sf * sum(c);
    if (a.square) y = fma(a.noise, a.V[(int64_t)(c0 + c) * a.ldv + ar], y);
    a.out[(int64_t)(c0 + c) * a.ldo + ar] = y;
  }
}

// out = s_f sum over the splits (in split order) + sigma^2 V, for the slab's rows.
__global__ __launch_bounds__(256) void fp64_splitsum_kernel(F64Args a, int64_t nsplit) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t row = a.row0 + r;
  const int c = blockIdx.y;
  if (r >= a.slab || row >= a.m) return;
  const double* src = a.part + (int64_t)c * a.slab + r;
  const int64_t step = (int64_t)a.t * a.slab;
  double s = 0.0;
  int64_t sp = 0;
  for (; sp + 8 <= nsplit; sp += 8, src += 8 * step) {  // eight loads in flight
    double v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = src[j * step];
#pragma unroll
    for (int j = 0; j < 8; ++j) s += v[j];
  }
  for (; sp < nsplit; ++sp, src += step) s += src[0];
  double y = a.sf * s;
  if (a.square) y = fma(a.noise, a.V[(int64_t)c * a.ldv + row], y);
  a.out[(int64_t)c * a.ldo + row] = y;
}

// How the FP64 form splits the b range.  Square products: until the grid has
// about kF64Groups workgroups (three rounds of the two that a CU holds), with at
// least kF64MinChunks chunks in a split.  Cross products: from n alone, so
// that a row's sums do not depend on the other rows of the call.  The partial
// sums are bounded by taking the rows in slabs and the columns in passes, such
// that a plan that needs no partials within GP_KMM_NOALLOC_MAX_BYTES stays within
// it with them; points beyond kF64SplitMaxN leave no room and take one split
// (their rows alone fill the chip).
// n = 8,192, t = 50: 128 workgroups on 256 CUs took 1.08 ms, 1,536 take 0.34 ms.
//
// kF64MinChunks matters below n = 6,000 only (d = 48, us, at least 4 / 8 / 12 / 16 / 24
// chunks): n = 1,200, t = 16: 32 / 44 / 50 / 63 / 101; n = 2,000, t = 50: 60 / 52 / 62 / 84 /
// 114; n = 4,096, t = 50: 145 / 123 / 134 / 109 / 148; n = 6,000, t = 50: 223 / 224 / 235 / 231 /
// 234.  No one value is best; 12 is within 1.3 of the best from n = 2,000 on.  The error is 2e-16
// to 6e-16 (rms) with all of 4 to 16.
constexpr int64_t kF64Groups = 1536;
constexpr int64_t kF64MinChunks = 12;
constexpr int64_t kF64CrossSplits = 64;
constexpr int kF64PassCols = 512;
constexpr int64_t kF64SplitMaxN = (40ll << 20) / 8;

F64Split f64_split(int64_t n, int64_t m, bool square, int t) {
  F64Split s;
  const int64_t nchunks = (n + kF64Chunk - 1) / kF64Chunk;
  const int64_t row_wgs = (m + kF64Rows - 1) / kF64Rows * ((t + kF64Cols - 1) / kF64Cols);
  const int64_t want = n > kF64SplitMaxN ? 1 : (square ? (kF64Groups + row_wgs - 1) / row_wgs : kF64CrossSplits);
  s.nsplit = std::max<int64_t>(1, std::min(want, nchunks / kF64MinChunks));
  s.cps = (nchunks + s.nsplit - 1) / s.nsplit;
  s.nsplit = (nchunks + s.cps - 1) / s.cps;
  s.slab = (m + kF64Rows - 1) / kF64Rows * kF64Rows;
  s.cpass = t;
  s.bytes = 0;
  if (s.nsplit > 1) {
    const int64_t cap = std::min<int64_t>(48ll << 20, (60ll << 20) - 8 * n);
    s.cpass = std::min(t, kF64PassCols);
    const int64_t per_row = s.nsplit * s.cpass * 8;
    s.slab = std::min(s.slab, std::max<int64_t>(kF64Rows, cap / per_row / kF64Rows * kF64Rows));
    s.bytes = (size_t)(s.slab * per_row);
  }
  return s;
}

// Whether one to four columns beyond whole blocks of 16 go to the VALU, whose sums have
// another order: not in a cross product of more than 64 columns, which takes one
// launch or two by the number of its rows, on which a row's bits must not depend.
static bool on_valu(int live, bool square, int t) {
  return live % 16 >= 1 && live % 16 <= 4 && (square || t <= kF64Cols);
}

// One launch of 64-column groups for all columns, the last group padded (true), or one
// for the whole groups and one in a smaller form for the rest: by the rounds of the 512
// workgroups that run at a time and a workgroup's time, in MFMAs per 16 x 32 tile.  The second
// launch waits for the first: n = 60, d = 48, t = 100 21 us in one launch, 41 in two.
static bool one_launch(int64_t gx, int64_t nsplit, int whole, int rest, int d, bool square, int t) {
  const int base = (d + 15) / 16 * 8 + 15;  // distances and profile
  const int64_t all = base + 32, part = base + (on_valu(rest, square, t) ? rest / 16 * 8 + 2 : (rest + 15) / 16 * 8);
  auto rounds = [](int64_t w) { return (w + 511) / 512; };
  return rounds(gx * nsplit * (whole + 1)) * all <= rounds(gx * nsplit * whole) * all + rounds(gx * nsplit) * part;
}

template <int DP, int KIND>
static void launch_fp64(int live, int first_col, dim3 grid, const F64Args& a, hipStream_t st) {
#define GPK_F64(NCB, REM) sweep_fp64_kernel<DP, KIND, NCB, REM><<<grid, 256, 0, st>>>(a, first_col, live)
  const bool valu = on_valu(live, a.square != 0, a.columns);
  switch (valu ? live / 16 : (live + 15) / 16) {
    case 0: GPK_F64(0, 4); break;
    case 1: valu ? GPK_F64(1, 4) : GPK_F64(1, 0); break;
    case 2: valu ? GPK_F64(2, 4) : GPK_F64(2, 0); break;
    case 3: valu ? GPK_F64(3, 4) : GPK_F64(3, 0); break;
    default: GPK_F64(4, 0); break;
  }
#undef GPK_F64
}

static hipError_t launch_columns(int kind, int d, int live, int first_col, dim3 grid, const F64Args& a,
                                 hipStream_t st) {
  const bool m52 = kind == GP_MATERN52;
#define GPK_F64(DP) \
  m52 ? launch_fp64<DP, GP_MATERN52>(live, first_col, grid, a, st) : launch_fp64<DP, GP_RBF>(live, first_col, grid, a, st)
  switch ((d + 15) / 16) {
    case 1: GPK_F64(16); break;
    case 2: GPK_F64(32); break;
    case 3: GPK_F64(48); break;
    case 4: GPK_F64(64); break;
    default: return hipErrorInvalidValue;
  }
#undef GPK_F64
  return hipGetLastError();
}

// Feature scales as profile_coordinate_scale(kind) / l_j, each rounded once: a
// common factor off by d would shift every u by u d (5e-15 of an entry at u = 16
// with the factor itself rounded, against 9e-16 for the sums).
static Scale make_scale64(const gp_kernel* kern) {
  constexpr long double kLog2e = 1.442695040888963407359924681001892137L;
  const long double c = kern->kind == GP_MATERN52 ? sqrtl(5.0L) * kLog2e : sqrtl(0.5L * kLog2e);
  Scale s{};
  for (int j = 0; j < kern->d; ++j) s.s[j] = (double)(c / (long double)kern->lengthscale[j]);
  return s;
}

hipError_t fp64_prepare(KmmPlan& p, const gp_kernel* kern, const double* X, const double* Z, hipStream_t st) {
  if (!X || (!p.square && !Z) || !p.sc64) return hipErrorInvalidValue;
  p.x64 = X;
  p.z64 = p.square ? X : Z;
  prep_fp64_kernel<<<(unsigned)((std::max<int64_t>(p.n, p.d) + kF64Block - 1) / kF64Block), kF64Block, 0, st>>>(
      X, p.n, p.d, make_scale64(kern), p.sc64, p.nb64);
  return hipGetLastError();
}

hipError_t fp64_sweep(const KmmPlan& p, const double* V, int64_t ldv, int t, double* out, int64_t ldo,
                      hipStream_t st) {
  if (!p.x64 || !p.z64 || !V || !out || t < 1 || t > p.tmax) return hipErrorInvalidValue;
  const F64Split& sp = p.f64;
  F64Args a{};
  a.Xb = p.x64;
  a.nb = p.nb64;
  a.Xa = p.z64;
  a.sc = p.sc64;
  a.n = p.n;
  a.m = p.m;
  a.ldv = ldv;
  a.ldo = ldo;
  a.cps = sp.cps;
  a.slab = sp.slab;
  a.d = p.d;
  a.square = p.square ? 1 : 0;
  a.columns = t;
  a.sf = p.sf;
  a.noise = p.noise;
  a.part = sp.nsplit > 1 ? p.part : nullptr;
  for (int c0 = 0; c0 < t; c0 += sp.cpass) {
    a.t = std::min(sp.cpass, t - c0);
    a.V = V + (int64_t)c0 * ldv;
    a.out = out + (int64_t)c0 * ldo;
    const int whole = a.t / kF64Cols, rest = a.t % kF64Cols;
    for (a.row0 = 0; a.row0 < p.m; a.row0 += sp.slab) {
      const int64_t rows = std::min(sp.slab, p.m - a.row0);
      const unsigned gx = (unsigned)((rows + kF64Rows - 1) / kF64Rows);
      hipError_t e = hipSuccess;
      const bool one = whole > 0 && rest > 0 && one_launch(gx, sp.nsplit, whole, rest, p.d, p.square, t);
      if (whole > 0)
        e = launch_columns(p.kind, p.d, kF64Cols, 0, dim3(gx, (unsigned)(whole + one), (unsigned)sp.nsplit), a, st);
      if (e == hipSuccess && rest > 0 && !one)
        e = launch_columns(p.kind, p.d, rest, whole * kF64Cols, dim3(gx, 1, (unsigned)sp.nsplit), a, st);
      if (e != hipSuccess) return e;
      if (a.part) {
        fp64_splitsum_kernel<<<dim3((unsigned)((rows + 255) / 256), (unsigned)a.t), 256, 0, st>>>(a, sp.nsplit);
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
    }
  }
  return hipSuccess;
}

}  // namespace gpk
