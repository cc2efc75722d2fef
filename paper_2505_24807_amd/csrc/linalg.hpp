// Small device kernels and the dense eigensolver wrapper used by the SCF and
// the Davidson iteration.
#pragma once

#include <rocblas/rocblas.h>

#include "common.hpp"

namespace seqx {

constexpr int kSmallDense = 256;  // largest n of the one-workgroup Cholesky kernel
constexpr int kEigMax = 512;      // largest n of the k-lowest eigensolver
// smallest n of it in eigh_lowest, also where all pairs are wanted: its four
// launches take 33 us at n = 11 (65 with one cluster of all eigenvalues), 43 (75)
// at 16, 52 (91) at 20 and 110 (164) at 48, Jacobi sweeps 39 at 10, 70 at 16, 102 at
// 20 and 472 at 48.  All pairs of a Gram matrix near the identity (one cluster) stay
// ahead of the library's divide and conquer up to kEigMax: 166 us against 974 at 49,
// 588 / 2152 at 128, 827 / 2124 at 129, 1886 / 6035 at 256, 5717 / 11305 at 512
constexpr int kEigMin = 13;
// largest n whose reduction stays in one workgroup: a step there costs 1.2 us at
// n = 64, 2.0 at 128 and 3.5 at 192 (instructions of 8 wavefronts on one compute
// unit) against 2.8-2.9 across compute units
constexpr int kEigOneGroup = 128;

// k lowest eigenpairs, 2 <= n <= kEigMax (eig_lowest.hip): A's columns 0..k-1
// and w; reads the lower triangle.  scratch holds eig_lowest_scratch(n, k) doubles.
// Above kEigOneGroup rows wavefronts of different compute units wait for each
// other's values, at most poll_limit rounds of polling; if that is not enough
// (other work holds the GPU), A is left as it was and info and status (optional,
// the same word as a double) are kEigGaveUp, else 0.
constexpr int kEigGaveUp = -1;
constexpr int kEigPollLimit = 1 << 20;  // about a second
size_t eig_lowest_scratch(int n, int k);
void launch_eig_lowest(hipStream_t st, int n, double* A, int lda, int k, double* w, double* scratch, int* info,
                       double* status, int poll_limit);
// The lowest eigenpairs of many small problems (eig_lowest.hip), one workgroup
// each for the reduction and one for every pair: problem m (of order n[m] <= ld
// <= 64, where active[m]) reads the lower triangle of A + m ld^2 and writes its
// min(n, kfew) lowest pairs to val + m ld and to columns of vec + m ld^2, or
// min(n, kcap) pairs where n + kfew > ld.  scratch_stride >=
// eig_batch_scratch(ld, kcap) doubles of scratch a problem.
constexpr int kEigBatchPairs = 32;  // largest kcap
struct EigBatch {
  int ld, kfew, kcap;
  long scratch_stride;
  const int *n, *active;
  const double* A;
  double *vec, *val, *scratch;
};
size_t eig_batch_scratch(int ld, int kcap);
void launch_eig_batch(hipStream_t st, int nprob, const EigBatch& b);
// lower Cholesky in one workgroup (small_dense.hip)
void launch_small_potrf(hipStream_t st, int n, double* A, int lda, int* info);

// Dense symmetric eigensolver / Cholesky on the device (rocSOLVER), FP64,
// column-major storage.  One instance per context stream.
class DenseSolver {
 public:
  explicit DenseSolver(hipStream_t st);
  ~DenseSolver();
  DenseSolver(const DenseSolver&) = delete;
  DenseSolver& operator=(const DenseSolver&) = delete;
  // eigenvalues ascending into w[n]; eigenvectors overwrite A (columns); status
  // (device, optional): the info word as a double
  void eigh(int n, double* A, int lda, double* w, double* status = nullptr);
  // the k lowest eigenpairs only: w[0..k), eigenvectors in columns 0..k-1 of A
  // (the rest of A is overwritten).  kEigMin <= n <= kEigMax runs on the
  // kernels of eig_lowest.hip; other n use eigh.  Reads the lower triangle.
  // The info word (also at status) must be checked: on kEigGaveUp A is as before the call, and the caller repeats it
  // with library = true (eigh, whose kernels do not wait for each other).
  void eigh_lowest(int n, double* A, int lda, int k, double* w, double* status = nullptr, bool library = false);
  // lower Cholesky factor in place (upper triangle untouched); info reports
  // the first non-positive pivot.  n <= kSmallDense runs as one workgroup.
  void potrf(int n, double* A, int lda);
  // device info word of the last eigh / potrf calls (0 = success); synchronises
  int info_eigh();
  int info_potrf();
  // enqueue the copy of both info words (eigh, potrf) to host memory on the
  // solver's stream, for a caller that synchronises the stream anyway
  void info_async(int* host2);
  // the device info words (eigh, potrf), for kernels that gather them
  const int* info_device() const { return info_.p; }

 private:
  rocblas_handle h_ = nullptr;
  hipStream_t st_;
  DBuf<double> work_, small_;
  DBuf<int> info_;
  // rounds of polling of eigh_lowest; SEQX_EIG_POLL_LIMIT at construction, for
  // tests of a reduction that gives up
  int poll_limit_ = kEigPollLimit;
};

// elementwise / reduction helpers (all ordered on `st`)
void fill(hipStream_t st, double* x, long n, double v);
void copy(hipStream_t st, double* dst, const double* src, long n);
// y = x rounded to nearest FP32
void to_float(hipStream_t st, long n, const double* x, float* y);
void transpose(hipStream_t st, int rows, int cols, const double* src, long lds, double* dst, long ldd);
// y = a*x + b*y
void axpby(hipStream_t st, long n, double a, const double* x, double b, double* y);
// out = max |x| (deterministic two-stage reduction); ws >= 1024 doubles
void max_abs(hipStream_t st, long n, const double* x, double* out, double* ws);
// E = X - X^T for a square n x n row-major X (commutator from F P)
void antisym(hipStream_t st, int n, const double* X, double* E);
void zero_upper_cm(hipStream_t st, int n, double* A, int lda);
// diagonal guess density: each atom's core charge spread over its AOs
void guess_density(hipStream_t st, int nao, const int* atom_of_ao, const int* slot, const void* elems, double* P);
// solve the (m+1) x (m+1) DIIS system for m coefficients, B (m x m, ld) given; single thread
void diis_coefficients(hipStream_t st, int m, const double* B, int ldb, double* c);

}  // namespace seqx
