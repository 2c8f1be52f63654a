// Rayleigh-Ritz support kernels (host launch wrappers).
#pragma once
#include <algorithm>

#include <vector>

#include "fb_internal.h"

namespace fb {

struct JacobiJob {
  int32_t m;
  int32_t pad_;
  c128* A;        // in: Hermitian matrix (destroyed)
  int64_t lda;
  c128* V;        // scratch m x m (rotations accumulate here)
  int64_t ldv;
  c128* W;        // out: eigenvectors, columns in ascending eigenvalue order
  int64_t ldw;
  double* w;      // out: eigenvalues ascending
  int32_t* order; // scratch m
  int32_t* sweeps;// out (may be null)
};

// Eigenvalues are ranked ascending, ties by column; a NaN ranks as an infinity, so
// that the ranks are a permutation whatever the values.
__device__ __forceinline__ double rank_key(double w) { return fmin(w, __builtin_inf()); }

int fill_zero(c128* p, int64_t rows, int64_t cols, int64_t ld, hipStream_t st);

// Q += sum_p w_p X_p over the (node, direction) solutions of one slice, in
// the order p = 0, 1, ... (real B: Q += 2 Re(w_p X_p)).
constexpr int kMaxPairs = 128;
struct AccJob {
  c128* Q;
  int64_t ldq;
  const c128* X[kMaxPairs];
  int64_t ldx;
  c128 w[kMaxPairs];
  int32_t np;
  int32_t m;
  int32_t acc_real;
  int32_t init;  // 1: Q starts from zero (the first pairs of a sum), not read
};
int accumulate_pairs(const AccJob* jobs_dev, int njobs, int64_t n, int max_m, hipStream_t st);
int gather_cols(const void* src, int64_t lds, bool real_src, c128* dst, int64_t ldd,
                int64_t rows, int cols, const int32_t* idx_dev, const double* scale_dev,
                hipStream_t st);
int store_cols(const c128* src, int64_t lds, void* dst, int64_t ldd, bool real_dst, int64_t rows,
               int cols, const int32_t* idx_dev, hipStream_t st);
int hermitize(c128* A, int m, int64_t lda, hipStream_t st);
int band_matmul(const Band& bd, const c128* X, int64_t ldx, c128* Y, int64_t ldy, int m,
                hipStream_t st);
size_t eig_resid_part_doubles(int64_t n, int m);
int eig_residuals(const Band& bd, const c128* X, int64_t ldx, const double* lam, int m,
                  double* part, double* res, hipStream_t st);
int launch_jacobi(int njobs, JacobiJob* jobs_dev, int max_sweeps, double tol, hipStream_t st);

// Parallel block Jacobi (many workgroups per matrix) for larger matrices:
// work holds block_jacobi_bytes(m) per job, dv_dev one device descriptor
// per job (kBjDescBytes), norms_dev 2 doubles per job.  Synchronises.
constexpr size_t kBjDescBytes = 128;
size_t block_jacobi_bytes(int m);
int block_jacobi(const std::vector<JacobiJob>& jobs, const JacobiJob* jobs_dev, char* work,
                 void* dv_dev, double* norms_dev, int max_sweeps, double tol, hipStream_t st);

// Hermitian eigensolver dispatch: matrices up to kSmallJacobi by the cyclic
// Jacobi, larger ones by block Jacobi.  The cyclic Jacobi runs on one
// workgroup per matrix or with a launch per round over the whole chip
// (rounds_pay says which), with the same bits.
constexpr int kSmallJacobi = 256;
constexpr int kRoundJacobi = 80;
// Whether a call whose largest matrix has maxm columns, with sum2 = sum of m^2
// over its matrices, takes a launch per round.  One workgroup per matrix needs a
// time of about maxm^3 whatever the number of matrices (up to the CUs); a
// round needs its launch and a share for every element of every matrix.  ms, by
// rounds against one workgroup each: 80 columns, 1 matrix 3.0 / 3.3, 8 3.2 /
// 3.3, 16 3.4 / 3.3, 128 8.5 / 4.3; 96 columns, 32 5.9 / 6.1, 64 7.5 / 6.1;
// 128 columns, 32 9.5 / 14, 64 16.4 / 15.8; 200 columns, 64 61 / 66, 128 122 /
// 92; one of 250 with 128 of 79 22 / 108.  The line fits the crossings (9
// matrices of 80 columns, 31 of 96, 52 of 128, 68 of 200); below kRoundJacobi
// columns the two are within 5 %.
bool rounds_pay(int maxm, int64_t sum2, int cus);
struct EigWork {
  char* bj = nullptr;       // block Jacobi buffers
  void* dv = nullptr;       // descriptors
  double* norms = nullptr;  // per-job norms
};
size_t eig_work_bytes(const std::vector<int>& ms);
void carve_eig_work(struct Arena& ar, const std::vector<int>& ms, EigWork& w);
int reduced_eig(std::vector<JacobiJob> jobs, JacobiJob* jobs_dev, const EigWork& w,
                int max_sweeps, double tol, hipStream_t st);
// 2-norms of the m columns of X (n x m, leading dimension ldx) into nrm (m
// doubles); the columns with nrm > thr * max(nrm) listed in idx (ascending)
// with scale = 1 / nrm, their number in *kept (all device memory)
int col_norm_keep(const c128* X, int64_t n, int64_t ldx, int m, double thr, double* nrm,
                  int32_t* idx, double* scale, int32_t* kept, hipStream_t st);
int gram_keep(const double* s, int m, double drop, int32_t* idx, double* scale, int32_t* kept,
              hipStream_t st);

}  // namespace fb
