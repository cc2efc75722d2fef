// One-workgroup Cholesky factorisation for the small subspace problems of the
// TDHF Davidson iteration (n <= 256).
#include <cmath>

#include "linalg.hpp"
#include "wave.hpp"

namespace seqx {

namespace {

constexpr int kNT = 1024;
constexpr int kNW = kNT / 64;
typedef double d4 __attribute__((ext_vector_type(4)));

// Lower Cholesky of an n x n block (n <= 256), left-looking by panels of kPB
// columns: the panel first takes the products of all columns before it (one
// 16 x 16 tile of the FP64 matrix cores a wavefront), then one wavefront factors
// its diagonal block in registers (row r in lane r) and a thread of its own
// solves every row below against it; info = first bad pivot (1-based) or 0.
// Latency bounds it: a panel has four barriers and reads the columns before it
// with many loads in flight.  Three barriers a column and a trailing update in
// memory took 28 us at n = 40, 147 at 150 and 359 at 256: now 24, 99 and 209.
constexpr int kPB = 16;

__global__ void __launch_bounds__(kNT) small_potrf_kernel(int n, double* __restrict__ A, int lda, int* info) {
  __shared__ double P[kSmallDense][kPB + 1];
  __shared__ double dinv[kPB];
  __shared__ int bad;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid == 0) bad = 0;
  __syncthreads();
  for (int j0 = 0; j0 < n; j0 += kPB) {
    const int nb = min(kPB, n - j0), m = n - j0;  // panel: rows j0 + r, r < m; columns j0 + q, q < nb
    for (int t = wave; 16 * t < m; t += kNW) {
      const int r16 = lane & 15, k4 = lane >> 4;
      const double* ar = A + min(j0 + 16 * t + r16, n - 1);  // rows past n and columns past nb are not used
      const double* br = A + min(j0 + r16, n - 1);
      d4 acc = {0, 0, 0, 0};
      for (int k0 = 0; k0 < j0; k0 += 16) {
        double x[4], y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const long k = static_cast<long>(k0 + 4 * u + k4) * lda;
          x[u] = ar[k];
          y[u] = br[k];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[u], y[u], acc, 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 16 * t + k4 + 4 * i;
        if (r16 <= r && r < m && r16 < nb) P[r][r16] = A[(j0 + r) + static_cast<long>(j0 + r16) * lda] - acc[i];
      }
    }
    __syncthreads();
    if (wave == 0) {
      double a[kPB];
#pragma unroll
      for (int q = 0; q < kPB; ++q) a[q] = (q <= lane && lane < nb) ? P[lane][q] : 0.0;
      int first = 0;
#pragma unroll
      for (int q = 0; q < kPB; ++q)
        if (q < nb && first == 0) {  // uniform
          const double piv = lane_value(a[q], q);
          if (!(piv > 0.0) || !isfinite(piv)) {
            first = j0 + q + 1;
          } else {
            const double d = sqrt(piv), inv = 1.0 / d;
            if (lane == 0) dinv[q] = inv;
            a[q] = lane == q ? d : a[q] * inv;
#pragma unroll
            for (int qq = q + 1; qq < kPB; ++qq) a[qq] -= a[q] * lane_value(a[q], qq);
          }
        }
#pragma unroll
      for (int q = 0; q < kPB; ++q)
        if (q <= lane && lane < nb) P[lane][q] = a[q];
      if (lane == 0) bad = first;
    }
    __syncthreads();
    if (bad) break;
    if (kPB + tid < m) {  // nb = kPB here
      double x[kPB];
#pragma unroll
      for (int q = 0; q < kPB; ++q) x[q] = P[kPB + tid][q];
#pragma unroll
      for (int q = 0; q < kPB; ++q) {
        x[q] *= dinv[q];
#pragma unroll
        for (int qq = q + 1; qq < kPB; ++qq) x[qq] -= x[q] * P[qq][q];
      }
#pragma unroll
      for (int q = 0; q < kPB; ++q) P[kPB + tid][q] = x[q];
    }
    __syncthreads();
    for (int q = wave; q < nb; q += kNW)
      for (int r = q + lane; r < m; r += 64) A[(j0 + r) + static_cast<long>(j0 + q) * lda] = P[r][q];
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
