// Internal interface of the FP64 solver kernels (blas.hip) used by the host
// orchestration (solver.cpp, predict.cpp, grad.hip).
#pragma once

#include "internal.h"

namespace gpk {

constexpr int64_t kDotBlocks = 1024;  // target blocks of the column reductions
constexpr int64_t kAtbBlocks = 256;   // target blocks of the tall-skinny A^T B products
constexpr uint64_t kEps1StreamOffset = 65536;

constexpr unsigned kStatusNotPD = 1u;
constexpr unsigned kStatusNonFinite = 2u;

inline uint64_t splitmix64_host(uint64_t x) {
  uint64_t z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

struct RowSplit {
  int64_t rows_per_blk;
  int64_t nblk;
};
RowSplit row_split(int64_t n, int64_t target_blocks);

// Device-resident per-column state of an mBCG run (arrays of s entries).
struct MbcgState {
  int s;
  double* gamma[2];   // r.z of the current residual (iterations alternate between the copies)
  double* gamma0;     // b^T P^{-1} b
  double* dpart;      // partial sums [block][column] (row_split(n, kDotBlocks)) of d.w,
  double* rpart;      // of ||r||^2 after the residual update
  double* gpart;      // and of r.z after the preconditioner step
  double *dsum, *rsum, *gsum;  // the sums themselves, where there are many partial sums
  double* alpha;      // current step sizes (copied to the host every iteration)
  double* beta;
  double* bnorm;      // ||b|| (holds ||b||^2 until init)
  double* relres;
  int* active[2];     // likewise alternating
  int* iters;
  int* num_active;
  unsigned* status;
};

struct Precond {
  int rank = 0;
  const double* L = nullptr;      // n x rank, ld n
  const double* Cchol = nullptr;  // rank x rank lower, column-major
  double noise = 0.0;
};

struct PivState {
  int64_t* piv;     // k pivots
  double* pivval;   // residual diagonal at each pivot
  int* rank;        // steps completed
  double* bval;     // block maxima of the residual diagonal, two buffers of pivchol_blocks(n)
  int64_t* bidx;    // and their rows
};

hipError_t coldot(const double* A, const double* B, int64_t n, int s, double* out, double* partial, hipStream_t st);
// The first pass of coldot: partial[block * s + c] over row_split(n, kDotBlocks).
hipError_t coldot_partials(const double* A, const double* B, int64_t n, int s, double* partial, hipStream_t st);
size_t atb_partial_doubles(int64_t n, int pa, int qb);
hipError_t atb(const double* A, int pa, const double* B, int qb, int64_t n, double* out, double* partial,
               hipStream_t st);
// atb with the row split into (at most) nblk blocks; partial holds nblk * pa * qb doubles.
hipError_t atb_n(const double* A, int pa, const double* B, int qb, int64_t n, double* out, double* partial,
                 int64_t nblk, hipStream_t st);
// Y = post (V + sign A C) for A (nrows x kk, column-major, lda), C (kk x s, row-major
// with row stride ldc), V (null: 0) and Y (nrows x s, column-major), s <= kTallMaxS.
// Y may alias A or V.  split_k: the sums over k in four parts (for few rows and
// long sums); otherwise the bits of a scalar FMA loop over ascending k.
constexpr int kTallMaxS = 64;
hipError_t tall_product(const double* A, int64_t lda, int64_t nrows, int kk, const double* C, int64_t ldc, int s,
                        double sign, double post, const double* V, int64_t ldv, double* Y, int64_t ldy,
                        bool split_k, hipStream_t st);
// Z = P^{-1} R for an n x s block.  Y: rank x s scratch; partial: atb scratch.
hipError_t precond_apply(const Precond& pc, const double* R, double* Z, int64_t n, int s, double* Y,
                         double* partial, hipStream_t st);
hipError_t launch_probes(const double* y, int64_t n, int t, const double* L, int k, double noise, uint64_t seed,
                         double* B, hipStream_t st);
hipError_t launch_copy(const double* src, double* dst, int64_t count, hipStream_t st);
hipError_t launch_zero_words(void* dst, int64_t words, hipStream_t st);  // 32-bit words
hipError_t launch_gemv_sub(const double* Q, int64_t n, int jn, const double* h, double* w, hipStream_t st);
hipError_t launch_scale_rsqrt(const double* src, const double* s2, int64_t n, double* dst, hipStream_t st);
hipError_t launch_bidiag_solve(double* QR, int64_t n, int K, const double* lm, hipStream_t st);
hipError_t launch_predict_finish(const double* P, int64_t m, int kc, double sf, double* mean, double* var,
                                 hipStream_t st);
hipError_t launch_fill(double* dst, double v, int64_t count, hipStream_t st);

hipError_t mbcg_launch_init(const MbcgState& s, hipStream_t st);
// Step cur of an iteration reads gamma[cur], active[cur] and writes the other copies
// (update_d).  dpart, rpart and gpart must hold their partial sums.
hipError_t mbcg_launch_update_ur(MbcgState s, int cur, const double* D, const double* W, double* U, double* R,
                                 int64_t n, hipStream_t st);
hipError_t mbcg_launch_update_d(MbcgState s, int cur, int j, double tol, const double* Z, double* D, int64_t n,
                                hipStream_t st);

int64_t pivchol_blocks(int64_t n);
hipError_t pivchol_launch_step(const double* X, int64_t n, const gp_kernel* kern, double* L, double* delta,
                               const PivState& ps, int m, double stop_below, hipStream_t st);

// Dense FP64 pieces on the matrix cores (exact.hip).  Row-major matrices.
// C (m x nn) = L B, L m x m lower triangular as dense_lower_inverse leaves it.
hipError_t dense_lower_times(int64_t m, int64_t nn, const double* L, int64_t ldl, const double* B, int64_t ldb,
                             double* C, int64_t ldc, hipStream_t st);
// C (m x m) = A A^T for A m x kk: the tiles on and below the diagonal.
hipError_t dense_gram(int64_t m, int64_t kk, const double* A, int64_t lda, double* C, int64_t ldc, double* scratch,
                      int64_t scratch_doubles, hipStream_t st);
// Doubles of the diagonal-block scratch of the two routines below.
size_t dense_dinv_doubles(int64_t n);
// In-place lower Cholesky factor of the symmetric n x n A (lower triangle read);
// the inverses of its 64 x 64 diagonal blocks into Dinv; *info (device, zeroed by
// the caller) receives 1 + the first non-positive pivot.
hipError_t dense_cholesky(double* A, int64_t n, int* info, double* Dinv, hipStream_t st);
// L <- L^{-1} in place for a lower Cholesky factor and its Dinv; W: n x n scratch.
// Zero above the diagonal inside the 128 x 128 diagonal tiles, unset beyond them.
hipError_t dense_lower_inverse(double* L, double* W, const double* Dinv, int64_t n, hipStream_t st);

// Host: e_1^T log(T) e_1 for the Lanczos tridiagonal of CG coefficients
// (alpha[j*stride], beta[j*stride], j < J).  Returns false if T is not
// positive definite or the eigen-iteration fails.
bool lanczos_log_quadrature(const double* alpha, const double* beta, int J, int stride, double* out);
// Host: eigenvalues (ascending not guaranteed) and first eigenvector components of a
// symmetric tridiagonal matrix (diag a[0..n-1], off-diagonal b[0..n-2]).
bool tridiag_eig_first(int n, double* a, double* b, double* z);
// Host: in-place lower Cholesky factor of the symmetric k x k matrix A (row-major);
// false if A is not positive definite.
bool host_cholesky(std::vector<double>& A, int k);
// Host: all eigenpairs of the dense symmetric n x n matrix A (row-major, destroyed):
// A = Q diag(w) Q^T, Q row-major with the eigenvectors as columns.  False if the
// iteration does not converge.
bool sym_eig(int n, std::vector<double>& A, std::vector<double>& w, std::vector<double>& Q);

}  // namespace gpk
