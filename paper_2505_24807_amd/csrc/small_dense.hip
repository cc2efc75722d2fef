// One-workgroup Cholesky factorisation for the small subspace problems of the
// TDHF Davidson iteration (n <= 256).
#include <cmath>

#include "linalg.hpp"
#include "wave.hpp"

namespace seqx {

namespace {

constexpr int kNT = 1024;
constexpr int kNW = kNT / 64;

// lower Cholesky of an n x n block (n <= 256), blocked by panels of kPB
// columns: the panel is factored in LDS, then the trailing lower triangle takes
// the panel's rank-kPB update in one pass; info = first bad pivot (1-based) or 0
constexpr int kPB = 16;

__global__ void __launch_bounds__(kNT) small_potrf_kernel(int n, double* __restrict__ A, int lda, int* info) {
  __shared__ double P[kSmallDense][kPB + 1];
  __shared__ int bad;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) bad = 0;
  __syncthreads();
  for (int j0 = 0; j0 < n; j0 += kPB) {
    const int nb = min(kPB, n - j0), m = n - j0;  // panel: rows j0 + r, r < m; columns j0 + q, q < nb
    for (int q = wave; q < nb; q += kNW)
      for (int r = q + lane; r < m; r += 64) P[r][q] = A[(j0 + r) + static_cast<long>(j0 + q) * lda];
    __syncthreads();
    for (int q = 0; q < nb; ++q) {
      if (tid == 0) {
        const double a = P[q][q];
        if (!(a > 0.0) || !isfinite(a)) bad = j0 + q + 1;
        else P[q][q] = sqrt(a);
      }
      __syncthreads();
      if (bad) break;
      const double inv = 1.0 / P[q][q];
      for (int r = q + 1 + tid; r < m; r += kNT) P[r][q] *= inv;
      __syncthreads();
      for (int qq = q + 1 + wave; qq < nb; qq += kNW)
        for (int r = qq + lane; r < m; r += 64) P[r][qq] -= P[r][q] * P[qq][q];
      __syncthreads();
    }
    if (bad) break;
    for (int q = wave; q < nb; q += kNW)
      for (int r = q + lane; r < m; r += 64) A[(j0 + r) + static_cast<long>(j0 + q) * lda] = P[r][q];
    for (int cl = nb + wave; cl < m; cl += kNW)
      for (int r = cl + lane; r < m; r += 64) {
        double sacc = 0.0;
#pragma unroll
        for (int q = 0; q < kPB; ++q)
          if (q < nb) sacc += P[r][q] * P[cl][q];
        A[(j0 + r) + static_cast<long>(j0 + cl) * lda] -= sacc;
      }
    __syncthreads();
  }
  if (tid == 0) info[0] = bad;
}

}  // namespace

void launch_small_potrf(hipStream_t st, int n, double* A, int lda, int* info) {
  hipLaunchKernelGGL(small_potrf_kernel, dim3(1), dim3(kNT), 0, st, n, A, lda, info);
  SEQX_LAUNCH_CHECK();
}

}  // namespace seqx
