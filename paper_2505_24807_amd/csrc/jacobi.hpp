// Symmetric eigensolver for small matrices held in LDS by one workgroup of
// NT threads (a power of two, at most 256): cyclic Jacobi with the round-robin (tournament) ordering, so each
// round rotates ne/2 disjoint index pairs at once (rows, then columns), with
// ne = n rounded up to even.  Used for the small Gram and collapse matrices of the single-molecule
// solver.
#pragma once

#include "common.hpp"
#include "wave.hpp"

namespace seqx {

constexpr int kJacobiMax = 48;  // largest n held in LDS (two 48 x 49 FP64 arrays)

struct JacobiLds {
  double A[kJacobiMax][kJacobiMax + 1];
  double Q[kJacobiMax][kJacobiMax + 1];
  double c[kJacobiMax / 2], s[kJacobiMax / 2];
  int p[kJacobiMax / 2], q[kJacobiMax / 2];
  int perm[kJacobiMax];
  int nact;  // stamp of the last round that rotated a pair
  double red[256];
};

// 1 / sqrt(x) and 1 / x, x > 0, from the hardware estimates (relative error
// 2^-23) and STEPS Newton-Raphson steps: two are FP64 to rounding
template <int STEPS>
__device__ __forceinline__ double rsqrt_newton(double x) {
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int i = 0; i < STEPS; ++i) y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
  return y;
}
template <int STEPS>
__device__ __forceinline__ double rcp_newton(double x) {
  double y = __builtin_amdgcn_rcp(x);
#pragma unroll
  for (int i = 0; i < STEPS; ++i) y = fma(y, fma(-x, y, 1.0), y);
  return y;
}

// On entry L.A holds the symmetric n x n matrix (n <= NMAX <= kJacobiMax).  On
// exit L.Q holds the eigenvectors as columns, diag(L.A) the eigenvalues, and
// L.perm the ascending order of the eigenvalues.  Sweeps stop when the
// off-diagonal sum of squares is below 1e-28 of the total (elements ~1e-14 of
// the largest; FP64 rounding keeps the sum near n * 1e-32 of the total) or
// after 40 sweeps.
// A round is a chain of LDS accesses, barriers and one rotation angle; its time
// hardly depends on n.  So the elements of a thread are worked out once, all
// loads of a round stand before its stores, the angle takes no division or
// square root of the library, and where one wavefront holds every 2 x 2 block
// (n <= 16) no barrier is left.  All pairs of a random matrix, with the launch:
// n = 10 48 -> 39 us, 16 82 -> 70, 32 236 -> 193, 48 623 -> 472.
template <int NT, int NMAX>
__device__ inline void jacobi_lds(int n, JacobiLds& L) {
  constexpr int kBlocks = (NMAX / 2 * (NMAX / 2) + NT - 1) / NT, kCols = (NMAX * (NMAX / 2) + NT - 1) / NT;
  for (int idx = threadIdx.x; idx < n * n; idx += NT) {
    const int i = idx / n, j = idx % n;
    L.Q[i][j] = (i == j) ? 1.0 : 0.0;
  }
  __syncthreads();
  const int ne = n + (n & 1), half = ne / 2;
  int b1[kBlocks], b2[kBlocks], qr[kCols], qk[kCols];  // this thread's blocks of A and column pairs of Q
#pragma unroll
  for (int e = 0; e < kBlocks; ++e) {
    const int it = threadIdx.x + NT * e;
    b1[e] = it < half * half ? it / half : -1;
    b2[e] = it < half * half ? it % half : 0;
  }
#pragma unroll
  for (int e = 0; e < kCols; ++e) {
    const int it = threadIdx.x + NT * e;
    qr[e] = it < n * half ? it / half : -1;
    qk[e] = it < n * half ? it % half : 0;
  }
  if (threadIdx.x == 0) L.nact = 0;  // seen by all after the first barrier of the sweep
  for (int sweep = 0; sweep < 40; ++sweep) {
    double off = 0.0, tot = 0.0;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane < n)
      for (int i = wv; i < n; i += NT / 64) {
        const double a2 = L.A[i][lane] * L.A[i][lane];
        tot += a2;
        if (i != lane) off += a2;
      }
    {  // both sums in one pass: wavefront sums, then the wavefronts in order
      off = wave_sum64(off);
      tot = wave_sum64(tot);
      if (lane == 0) {
        L.red[2 * wv] = off;
        L.red[2 * wv + 1] = tot;
      }
      __syncthreads();
      off = 0.0;
      tot = 0.0;
      for (int q = 0; q < NT / 64; ++q) {
        off += L.red[2 * q];
        tot += L.red[2 * q + 1];
      }
      __syncthreads();
    }
    if (!(off > 1e-28 * tot)) break;
    // pairs whose element is below this are left alone: together they stay
    // two orders under the stopping bar (threshold Jacobi)
    const double skip2 = 1e-30 * tot / (static_cast<double>(n) * n);
    for (int r = 0; r < ne - 1; ++r) {
      const int stamp = sweep * ne + r + 1;  // unique per round: no reset needed
      if (threadIdx.x < half) {
        const int k = threadIdx.x;
        int p = r + k, q = r - k;
        if (p >= ne - 1) p -= ne - 1;
        if (q < 0) q += ne - 1;
        if (k == 0) q = ne - 1;
        if (p > q) { const int t = p; p = q; q = t; }
        double c = 1.0, s = 0.0;
        const double apq = q < n ? L.A[p][q] : 0.0;
        if (apq * apq > skip2) {
          // tan of the rotation, sign(d) a_pq / (|d| + sqrt(d^2 + a_pq^2)) with d half
          // the difference of the diagonal elements; only c must be exact, as then
          // c^2 + s^2 = 1
          const double d = 0.5 * (L.A[q][q] - L.A[p][p]), h = fma(d, d, apq * apq);
          const double t = (d >= 0.0 ? apq : -apq) * rcp_newton<1>(fabs(d) + h * rsqrt_newton<1>(h));
          c = rsqrt_newton<2>(fma(t, t, 1.0));
          s = t * c;
          L.nact = stamp;  // benign race: every writer stores the same value
        } else if (q >= n) {
          q = p;  // the spare index of odd n: identity rotation of p onto itself (p is in no other pair)
        }  // a pair left alone keeps both indices with the identity rotation, so
           // that every index still belongs to one pair of the round
        L.p[k] = p;
        L.q[k] = q;
        L.c[k] = c;
        L.s[k] = s;
      }
      __syncthreads();
      if (L.nact != stamp) continue;  // uniform: nothing to rotate in this round
      // The pairs of a round are disjoint, so A' = J^T A J splits into 2 x 2
      // blocks (rows of pair k1, columns of pair k2), each formed from its own
      // four elements, and Q' = Q J into pairs of columns: one pass and one
      // barrier.  The pairs cover every index once (the spare slot of odd n
      // as q = p, which reads and writes one element several times with the
      // same value).
      double x[kBlocks][4], y[kCols][2];
      int ap[kBlocks][4], qp[kCols][2];  // positions in A and Q
      double* A = &L.A[0][0];
      double* Q = &L.Q[0][0];
      constexpr int ld = kJacobiMax + 1;
#pragma unroll
      for (int e = 0; e < kBlocks; ++e)
        if (b1[e] >= 0) {
          const int p1 = L.p[b1[e]], q1 = L.q[b1[e]], p2 = L.p[b2[e]], q2 = L.q[b2[e]];
          ap[e][0] = p1 * ld + p2;
          ap[e][1] = p1 * ld + q2;
          ap[e][2] = q1 * ld + p2;
          ap[e][3] = q1 * ld + q2;
#pragma unroll
          for (int i = 0; i < 4; ++i) x[e][i] = A[ap[e][i]];
          const double c1 = L.c[b1[e]], s1 = L.s[b1[e]], c2 = L.c[b2[e]], s2 = L.s[b2[e]];
          // rows p1, q1 first (columns p2 and q2), then columns p2, q2
          const double bpp = c1 * x[e][0] - s1 * x[e][2], bqp = s1 * x[e][0] + c1 * x[e][2];
          const double bpq = c1 * x[e][1] - s1 * x[e][3], bqq = s1 * x[e][1] + c1 * x[e][3];
          x[e][0] = c2 * bpp - s2 * bpq;
          x[e][1] = s2 * bpp + c2 * bpq;
          x[e][2] = c2 * bqp - s2 * bqq;
          x[e][3] = s2 * bqp + c2 * bqq;
        }
#pragma unroll
      for (int e = 0; e < kCols; ++e)
        if (qr[e] >= 0) {
          qp[e][0] = qr[e] * ld + L.p[qk[e]];
          qp[e][1] = qr[e] * ld + L.q[qk[e]];
          const double c2 = L.c[qk[e]], s2 = L.s[qk[e]];
          const double vp = Q[qp[e][0]], vq = Q[qp[e][1]];
          y[e][0] = c2 * vp - s2 * vq;
          y[e][1] = s2 * vp + c2 * vq;
        }
#pragma unroll
      for (int e = 0; e < kBlocks; ++e)
        if (b1[e] >= 0)
#pragma unroll
          for (int i = 0; i < 4; ++i) A[ap[e][i]] = x[e][i];
#pragma unroll
      for (int e = 0; e < kCols; ++e)
        if (qr[e] >= 0)
#pragma unroll
          for (int i = 0; i < 2; ++i) Q[qp[e][i]] = y[e][i];
      __syncthreads();
    }
  }
  // ascending order, stable: eigenvalue i goes to the place given by how many
  // eigenvalues lie below it (ties by index), all ranks at once.  perm starts
  // as the identity, so it only ever holds valid indices (NaNs would collide).
  for (int i = threadIdx.x; i < n; i += NT) L.perm[i] = i;
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += NT) {
    const double li = L.A[i][i];
    int r = 0;
    for (int j = 0; j < n; ++j) {
      const double lj = L.A[j][j];
      r += (lj < li || (lj == li && j < i)) ? 1 : 0;
    }
    if (r < n) L.perm[r] = i;
  }
  __syncthreads();
}

}  // namespace seqx
