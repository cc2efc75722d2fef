// Pulay (DIIS) coefficients of the SCF, solved by one workgroup.
#pragma once

#include <hip/hip_runtime.h>

namespace seqx {

constexpr int kDiisMax = 16;  // longest history

struct DiisLds {
  double a[kDiisMax + 1][kDiisMax + 3], sc;
  int piv;
};

// Coefficients c[0 .. m) of m error overlaps B (leading dimension ldb): Gauss-
// Jordan with partial pivoting on the bordered system, one row per thread (at
// least m + 2 threads; every thread of the workgroup calls).  A singular system
// falls back to the newest matrix only.  Ends with a barrier after c is written.
__device__ inline void diis_solve(int m, const double* B, int ldb, double* c, DiisLds& L) {
  const int t = threadIdx.x, n = m + 1;
  if (t < m) {
    for (int j = 0; j < m; ++j) L.a[t][j] = B[t * ldb + j];
    L.a[t][m] = -1.0;
    L.a[t][n] = 0.0;
  } else if (t == m) {
    for (int j = 0; j < m; ++j) L.a[m][j] = -1.0;
    L.a[m][m] = 0.0;
    L.a[m][n] = -1.0;
  }
  __syncthreads();
  if (t == 0) {  // scale the error block for conditioning
    double sc = 0.0;
    for (int i = 0; i < m; ++i) sc = fmax(sc, fabs(L.a[i][i]));
    L.sc = sc;
  }
  __syncthreads();
  if (L.sc > 0 && t < m)
    for (int j = 0; j < m; ++j) L.a[t][j] /= L.sc;
  __syncthreads();
  bool singular = false;
  for (int col = 0; col < n; ++col) {
    if (t == 0) {
      int piv = col;
      for (int r = col + 1; r < n; ++r)
        if (fabs(L.a[r][col]) > fabs(L.a[piv][col])) piv = r;
      L.piv = piv;
    }
    __syncthreads();
    const int piv = L.piv;
    if (piv != col && t <= n) {  // column t of the two rows
      const double tmp = L.a[col][t];
      L.a[col][t] = L.a[piv][t];
      L.a[piv][t] = tmp;
    }
    __syncthreads();
    const double d = L.a[col][col];
    if (d == 0.0) {  // the same in every thread
      singular = true;
      break;
    }
    if (t < n && t != col) {
      const double f = L.a[t][col] / d;
      for (int j = col; j <= n; ++j) L.a[t][j] -= f * L.a[col][j];
    }
    __syncthreads();
  }
  if (t < m) c[t] = singular ? (t == m - 1 ? 1.0 : 0.0) : L.a[t][n] / L.a[t][t];
  __syncthreads();
}

}  // namespace seqx
