// The k lowest eigenpairs of a dense symmetric matrix of at most 512 rows (the
// projected problems of the Davidson iteration), as four kernels:
//   1. Householder reduction to tridiagonal form T = Q^T A Q;
//   2. one workgroup per eigenpair: the eigenvalue by Sturm-count multisection
//      (256 points a round), the eigenvector of T by inverse iteration;
//   3. Gram-Schmidt inside clusters of close eigenvalues;
//   4. one wavefront per vector: y = Q z.
// All of them are chains of n dependent steps, so what counts is the latency
// of a step, not its few thousand operations: vectors live in registers, one
// element per lane and 64-row block, scalars of a step come by lane reads, and
// sums over a vector are lane moves.
//
// Time for 10 pairs (random matrix): n = 64 142 us, 128 390, 240 955, 440
// 2260; one workgroup for everything with the block lower triangle in registers
// took 1720 at n = 240, and a library divide-and-conquer solve about 5300 at
// n = 440.  Of the 955 us, 697 are the reduction (2.9 us a step, most of it the
// exchange through memory), 217 the pairs of T, 84 the back-transformation.  20
// CIS roots of C40H42: 130 -> 51 ms; the mixed (H2O)330 TDHF step 992 -> 937 ms.
#include <cmath>

#include "linalg.hpp"
#include "wave.hpp"

namespace seqx {

namespace {

// arr[c] for a uniform c without indexing registers dynamically
template <int NC>
__device__ __forceinline__ double pick(const double (&arr)[NC], int c) {
  double r = arr[0];
#pragma unroll
  for (int q = 1; q < NC; ++q) r = c == q ? arr[q] : r;
  return r;
}

// element i (uniform) of a vector held one element per lane and block
template <int NC>
__device__ __forceinline__ double element(const double (&arr)[NC], int i) {
  return lane_value(pick<NC>(arr, i >> 6), i & 63);
}

// element wave + NW k of such a vector, with the block known at compile time
// where the wavefront count allows it
template <int NC, int NW>
__device__ __forceinline__ double row_element(const double (&arr)[NC], int wave, int k) {
  const int i = wave + NW * k;
  if constexpr (NW <= 64 && 64 % NW == 0) return lane_value(arr[NW * k >> 6], i & 63);
  return element<NC>(arr, i);
}

// workgroup barrier that orders LDS accesses only
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// 1 / x from the hardware reciprocal estimate and one Newton-Raphson step
// (x finite and nonzero)
__device__ __forceinline__ double rcp_nr(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  return fma(r, fma(-x, r, 1.0), r);
}

// ---------------------------------------------------------------- 1. tridiagonal form

// A value not yet published in the exchange area: a NaN that no arithmetic makes
// of numbers.  (One that came with the input keeps its bits through arithmetic:
// it is published as another NaN.)
constexpr unsigned long long kEmpty = ~0ull;
__global__ void __launch_bounds__(256) exchange_fill_kernel(long n, unsigned long long* __restrict__ x, int* failed) {
  const long i = blockIdx.x * 256L + threadIdx.x;
  if (i < n) x[i] = kEmpty;
  if (i == 0) *failed = 0;
}

__device__ __forceinline__ void publish(double* p, double v) {
  const unsigned long long b = static_cast<unsigned long long>(__double_as_longlong(v));
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), b == kEmpty ? kEmpty >> 1 : b, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long peek(const double* p) {
  return __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// NW wavefronts hold the full symmetric matrix in registers: wavefront w keeps
// rows w, w + NW, ... (NR of them), lane l the columns l + 64 c (NC blocks).
// Step j: every wavefront forms the reflector of column j from its own copy of
// the column (the same operations everywhere, so the copies agree bit for
// bit), multiplies its rows with it, and the wavefronts exchange p = A v and
// row j + 1 once; then each forms w = tau p - (tau^2 v^T p / 2) v, the next
// column from the exchanged row, and updates its rows by -v w^T - w v^T.  One
// exchange a step is all the communication.
//
// GRID = false: one workgroup, exchange through LDS (one barrier a step; two
// LDS copies in turn).  GRID = true: wavefronts on different compute units,
// exchange through memory: every value has a place of its own that holds kEmpty
// until it is stored, so a reader simply polls the values it needs (device
// scope; no counter, no ordering between values).  The grid is at most 64
// single-wavefront workgroups, which are resident together unless other work
// holds the GPU: a wavefront that has polled poll_limit rounds (about a second at
// kEigPollLimit) gives up, so every wait ends.  The matrix is then left as it
// was and the caller told (kEigGaveUp).
template <int NC, int NR, int NW, bool GRID>
__device__ __forceinline__ void tridiagonalise(int n, const double* __restrict__ A, int lda, double* __restrict__ W,
                                               double* __restrict__ dte, double* xch, int* failed,
                                                int poll_limit) {
  static_assert(NW * NR >= 64 * NC, "rows must be covered");
  __shared__ double sp[2][GRID ? 1 : 64 * NC], sy[2][GRID ? 1 : 64 * NC];
  const int lane = threadIdx.x & 63;
  const int wave = GRID ? static_cast<int>(blockIdx.x) : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double* dd = dte;
  double* ee = dte + n;
  double* tt = dte + 2 * n;
  double a[NR][NC], x[NC];
#pragma unroll
  for (int k = 0; k < NR; ++k)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int l = wave + NW * k, i = lane + 64 * c;
      const int r = i > l ? i : l, s = i > l ? l : i;  // read the lower triangle
      a[k][c] = (l < n && i < n) ? A[r + static_cast<long>(s) * lda] : 0.0;
    }
#pragma unroll
  for (int c = 0; c < NC; ++c) x[c] = lane + 64 * c < n ? A[lane + 64 * c] : 0.0;
  for (int j = 0; j + 2 < n; ++j) {
    // reflector H = I - t v v^T with H x = alpha e_1, x = column j below the diagonal
    double xsq = 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const double xi = lane + 64 * c > j ? x[c] : 0.0;
      xsq += xi * xi;
    }
    const double xx = wave_sum64(xsq);
    const double x0 = element<NC>(x, j + 1);
    double alpha = 0.0, v0 = x0, t = 0.0;
    if (xx > 0.0) {
      alpha = x0 > 0.0 ? -sqrt(xx) : sqrt(xx);
      v0 = x0 - alpha;
      t = 2.0 / (xx - x0 * x0 + v0 * v0);
    }
    double v[NC];  // zero at rows <= j
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int i = lane + 64 * c;
      v[c] = i == j + 1 ? v0 : (i > j + 1 ? x[c] : 0.0);
    }
    if (wave == 0) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int i = lane + 64 * c;
        if (i > j && i < n) W[static_cast<long>(j) * n + i] = v[c];
        if (i == j) dd[j] = x[c];
      }
      if (lane == 0) {
        ee[j] = alpha;
        tt[j] = t;
      }
    }
    // this wavefront's elements of p = A v, and row j + 1 from its owner
    double* spj = sp[j & 1];
    double* syj = sy[j & 1];
    double* xp = xch + 2L * j * n;
    double* xy = xp + n;
    if ((j + 1) % NW == wave) {
      const int ko = (j + 1) / NW;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        double y = a[0][c];
#pragma unroll
        for (int k = 1; k < NR; ++k) y = ko == k ? a[k][c] : y;
        const int i = lane + 64 * c;
        if (i > j && i < n) {
          if constexpr (GRID) publish(xy + i, y);
          else syj[i] = y;
        }
      }
    }
    if constexpr (GRID) {
      double mine = 0.0;
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        const int i = wave + NW * k;
        if (i > j && i < n) {  // uniform
          double s = 0.0;
#pragma unroll
          for (int c = 0; c < NC; ++c) s += a[k][c] * v[c];
          s = wave_sum64(s);
          mine = lane == k ? s : mine;
        }
      }
      const int i = wave + NW * lane;
      if (lane < NR && i > j && i < n) publish(xp + i, mine);
    } else {
#pragma unroll
      for (int q = 0; q < NR / 8; ++q) {
        if (wave + NW * (8 * q + 7) > j && wave + NW * 8 * q < n) {  // uniform: a row of the eight is active
          double cs[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            cs[u] = 0.0;
#pragma unroll
            for (int c = 0; c < NC; ++c) cs[u] += a[8 * q + u][c] * v[c];
          }
          const double cl = wave_sum8x64(cs);  // row u = (lane >> 3) & 7
          const int i = wave + NW * (8 * q + (lane >> 3));
          if ((lane & 7) == 0 && i > j && i < n) spj[i] = cl;
        }
      }
    }
    double p[NC], y[NC];
    if constexpr (GRID) {
      for (int round = 0;; ++round) {
        bool ready = true;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const int i = lane + 64 * c;
          const bool need = i > j && i < n;
          const unsigned long long bp = need ? peek(xp + i) : 0ull, by = need ? peek(xy + i) : 0ull;
          ready = ready && bp != kEmpty && by != kEmpty;
          p[c] = __longlong_as_double(static_cast<long long>(bp));
          y[c] = __longlong_as_double(static_cast<long long>(by));
        }
        if (__all(ready)) break;
        if (round >= poll_limit) {
          if (lane == 0) *failed = 1;
          return;
        }
      }
    } else {
      lds_barrier();
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int i = lane + 64 * c;
        const bool need = i > j && i < n;
        p[c] = need ? spj[i] : 0.0;
        y[c] = need ? syj[i] : 0.0;
      }
    }
    double vp = 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c) vp += v[c] * p[c];
    const double K = 0.5 * t * t * wave_sum64(vp);
    double w[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) w[c] = t * p[c] - K * v[c];
    const double w1 = element<NC>(w, j + 1);
#pragma unroll
    for (int c = 0; c < NC; ++c) x[c] = fma(-w[c], v0, fma(-v[c], w1, y[c]));
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const int i = wave + NW * k;
      if (i > j + 1 && i < n) {  // uniform
        const double vi = row_element<NC, NW>(v, wave, k), wi = row_element<NC, NW>(w, wave, k);
#pragma unroll
        for (int c = 0; c < NC; ++c) a[k][c] = fma(-w[c], vi, fma(-v[c], wi, a[k][c]));
      }
    }
  }
  // the last 2 x 2 block
  if (wave == 0) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int i = lane + 64 * c;
      if (i == n - 2) {
        dd[i] = x[c];
        tt[i] = 0.0;
      }
      if (i == n - 1) {
        ee[n - 2] = x[c];
        ee[i] = 0.0;
        tt[i] = 0.0;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < NR; ++k)
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (wave + NW * k == n - 1 && lane + 64 * c == n - 1) dd[n - 1] = a[k][c];
}

template <int NC, int NR, int NW, bool GRID>
__global__ void __launch_bounds__(GRID ? 64 : 64 * NW) tridiag_kernel(int n, const double* __restrict__ A, int lda,
                                                                      double* __restrict__ W,
                                                                      double* __restrict__ dte, double* xch,
                                                                      int* failed, int poll_limit) {
  tridiagonalise<NC, NR, NW, GRID>(n, A, lda, W, dte, xch, failed, poll_limit);
}

// ---------------------------------------------------------------- 2. eigenpairs of T

// number of eigenvalues of T (d, e2 = e^2) below x: the sign changes of the
// leading principal minors p_i = (d_i - x) p_{i-1} - e2_{i-1} p_{i-2} of T - x I,
// a multiply and a fused multiply-add a step where the quotients of the LDL^T
// factorisation would divide.  A zero minor counts as a change and is replaced
// by a tiny one of that sign, so that the sequence goes on behind it (T may
// split there).  Every 8 steps both minors are scaled by one power of two (exact).
__device__ int sturm_count(int n, const double* d, const double* e2, double x) {
  int c = 0;
  double pp = 0.0, p = 1.0;  // p_{i-2}, p_{i-1} (p_{-1} = 1)
  auto step = [&](double dx, double f) {  // selects, no branches
    const double pn = fma(dx, p, -f * pp);
    const double q = pn == 0.0 ? -0x1p-60 * p : pn;
    c += static_cast<int>(static_cast<unsigned>(__double2hiint(q) ^ __double2hiint(p)) >> 31);
    pp = p;
    p = q;
  };
  int i = 0;
  for (; i + 8 <= n; i += 8) {
    double dx[8], f[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      dx[u] = d[i + u] - x;
      f[u] = e2[i + u];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) step(dx[u], f[u]);
    const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(pp)));
    p = ldexp(p, -ex);
    pp = ldexp(pp, -ex);
  }
  for (; i < n; ++i) step(d[i] - x, e2[i]);
  return c;
}

// 256 points a round (one wavefront per SIMD): the count is bound by its
// instructions, and 512 points took twice the time for one round less in seven
constexpr int kPairThreads = 256;

// eigenpair tt: lam[tt], Z[tt * n ..]; the workgroup of pair 0 also stores |T|
template <int NC>
__device__ __forceinline__ void tridiag_pair(int tt, int n, const double* __restrict__ dte, double* __restrict__ lam,
                                             double* __restrict__ Z, double* __restrict__ norm) {
  __shared__ double d[64 * NC], e2[64 * NC];  // e2[i] = e_{i-1}^2
  __shared__ int first[2][kPairThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  double dr[NC], er[NC];  // d_i and e_i of rows lane + 64 c (e_{n-1} = 0)
  double lo = 1e300, hi = -1e300;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int i = lane + 64 * c;
    dr[c] = i < n ? dte[i] : 0.0;
    er[c] = i + 1 < n ? dte[n + i] : 0.0;
    if (i < n) {
      const double el = i > 0 ? fabs(dte[n + i - 1]) : 0.0, r = el + fabs(er[c]);
      lo = fmin(lo, dr[c] - r);
      hi = fmax(hi, dr[c] + r);
      if (wave == 0) {
        d[i] = dr[c];
        e2[i] = el * el;
      }
    }
  }
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
    lo = fmin(lo, __shfl_xor(lo, m));
    hi = fmax(hi, __shfl_xor(hi, m));
  }
  __syncthreads();
  const double tnorm = fmax(fabs(lo), fabs(hi));
  if (tt == 0 && tid == 0) *norm = tnorm;
  double a = lo - (2.2e-16 * tnorm * n + 1e-300), b = hi + (2.2e-16 * tnorm * n + 1e-300);
  constexpr double fold = kPairThreads + 1;
  for (int round = 0; round < 40; ++round) {
    if (!(b - a > 4.4e-16 * fmax(fabs(a), fabs(b)) + 1e-300)) break;  // uniform
    const double x = a + (b - a) * (tid + 1) / fold;
    // first point with more than tt eigenvalues below it
    const unsigned long long above = __ballot(sturm_count(n, d, e2, x) > tt);
    int* f = first[round & 1];
    if (lane == 0) f[wave] = above ? 64 * wave + __ffsll(static_cast<long long>(above)) - 1 : kPairThreads;
    lds_barrier();
    int k = kPairThreads;
#pragma unroll
    for (int q = 0; q < kPairThreads / 64; ++q) k = min(k, f[q]);
    const double na = k == 0 ? a : a + (b - a) * k / fold;
    const double nb = k == kPairThreads ? b : a + (b - a) * (k + 1) / fold;
    a = na;
    b = nb;
  }
  const double l_t = 0.5 * (a + b);
  if (tid == 0) lam[tt] = l_t;
  if (wave != 0) return;
  // Inverse iteration by one wavefront: P (T - lam I) = L U with two
  // superdiagonals in U; row i of U is (1 / u0, u1, u2), lm the multipliers.
  // Multipliers and pivots come from reciprocals (one Newton step on the
  // hardware estimate): the factorisation only needs to be that of a nearby matrix.
  const double pert = 2.2e-16 * tnorm + 1e-300;
  double u0[NC], u1[NC], u2[NC], lm[NC], y[NC];
  bool sw[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    u0[c] = u1[c] = u2[c] = lm[c] = 0.0;
    sw[c] = false;
    // deterministic start: a fixed pseudo-random vector per eigenvalue index
    unsigned long long s = (static_cast<unsigned long long>(tt + 1) << 32) + static_cast<unsigned>(lane + 64 * c);
    s = (s + 0x9E3779B97F4A7C15ULL) * 0xBF58476D1CE4E5B9ULL;
    s ^= s >> 27;
    s *= 0x94D049BB133111EBULL;
    s ^= s >> 31;
    y[c] = lane + 64 * c < n ? static_cast<double>(s >> 11) / 9007199254740992.0 - 0.5 : 0.0;
  }
  double c0 = lane_value(dr[0], 0) - l_t, c1 = lane_value(er[0], 0);  // current pivot row
  double c2 = 0.0;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int cn = c + 1 < NC ? c + 1 : c;
    const int m = min(64, n - 1 - 64 * c);
    for (int l = 0; l < m; ++l) {
      const double sub = lane_value(er[c], l);
      const double dn = l < 63 ? lane_value(dr[c], l + 1) : lane_value(dr[cn], 0);
      const double r2 = l < 63 ? lane_value(er[c], l + 1) : lane_value(er[cn], 0);
      const double r1 = dn - l_t;
      const bool swap = fabs(sub) > fabs(c0);
      const double piv = swap ? sub : c0, oth = swap ? c0 : sub;
      const double q1 = swap ? r1 : c1, q2 = swap ? r2 : c2;    // pivot row beyond the pivot
      const double s1 = swap ? c1 : r1, s2 = swap ? c2 : r2;    // the other row
      const double safe = fabs(piv) < pert ? (piv < 0.0 ? -pert : pert) : piv;
      const double mlt = piv != 0.0 ? oth * rcp_nr(piv) : 0.0;
      const bool me = lane == l;
      u0[c] = me ? rcp_nr(safe) : u0[c];
      u1[c] = me ? q1 : u1[c];
      u2[c] = me ? q2 : u2[c];
      lm[c] = me ? mlt : lm[c];
      sw[c] = me ? swap : sw[c];
      c0 = fma(-mlt, q1, s1);
      c1 = fma(-mlt, q2, s2);
      c2 = 0.0;
    }
  }
  {
    const double safe = fabs(c0) < pert ? (c0 < 0.0 ? -pert : pert) : c0, r = rcp_nr(safe);
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (lane + 64 * c == n - 1) {
        u0[c] = r;
        u1[c] = 0.0;
        u2[c] = 0.0;
      }
  }
  for (int it = 0; it < 2; ++it) {
    if (it > 0) {  // the start vector stands for P L^-1 of a random one
    double carry = lane_value(y[0], 0);  // running element i of P L^-1 y
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int cn = c + 1 < NC ? c + 1 : c;
      const int m = min(64, n - 1 - 64 * c);
      const unsigned long long swm = __ballot(sw[c]);
      for (int l = 0; l < m; ++l) {
        const double nx = l < 63 ? lane_value(y[c], l + 1) : lane_value(y[cn], 0);
        const double ml = lane_value(lm[c], l);
        const bool s = (swm >> l) & 1;
        const double yi = s ? nx : carry, ot = s ? carry : nx;
        y[c] = lane == l ? yi : y[c];
        carry = fma(-ml, yi, ot);
      }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) y[c] = lane + 64 * c == n - 1 ? carry : y[c];
    }
    double x1 = 0.0, x2 = 0.0;  // solution at rows i + 1, i + 2
#pragma unroll
    for (int c = NC - 1; c >= 0; --c)
      for (int l = min(63, n - 1 - 64 * c); l >= 0; --l) {
        const double yv = lane_value(y[c], l), a0 = lane_value(u0[c], l);
        const double a1 = lane_value(u1[c], l), a2 = lane_value(u2[c], l);
        const double xi = fma(-a1, x1, fma(-a2, x2, yv)) * a0;
        y[c] = lane == l ? xi : y[c];
        x2 = x1;
        x1 = xi;
      }
    double nrm = 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c) nrm += y[c] * y[c];
    const double inv = 1.0 / sqrt(wave_sum64(nrm));
#pragma unroll
    for (int c = 0; c < NC; ++c) y[c] *= inv;
  }
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (lane + 64 * c < n) Z[static_cast<long>(tt) * n + lane + 64 * c] = y[c];
}

template <int NC>
__global__ void __launch_bounds__(kPairThreads) tridiag_pair_kernel(int n, const double* __restrict__ dte,
                                                                    double* __restrict__ lam,
                                                                    double* __restrict__ Z,
                                                                    double* __restrict__ norm) {
  tridiag_pair<NC>(blockIdx.x, n, dte, lam, Z, norm);
}

// ---------------------------------------------------------------- 3. clusters

constexpr int kClusterThreads = 1024;
constexpr int kClusterLds = 16384;  // eigenvector elements staged in LDS

// Orthogonalisation inside clusters of close eigenvalues (|lam_s - lam_t| <
// 1e-3 |T|): vector t against the cluster members s < t, in order of t, two
// classical Gram-Schmidt passes (one wavefront per inner product).  Vectors
// are staged in LDS when they fit, else stay in memory.
template <bool STAGED, int NT, int LDS, int KMAX>
__device__ __forceinline__ void orthogonalise_clusters(int n, int k, const double* __restrict__ lam,
                                                       const double* __restrict__ norm, double* Z) {
  __shared__ double stage[STAGED ? LDS : 1];
  __shared__ double red[KMAX];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const double gap = 1e-3 * *norm;
  // eigenvalues ascend: without a close pair of neighbours there is no cluster
  bool any = false;
  for (int t = 1; t < k; ++t) any = any || fabs(lam[t - 1] - lam[t]) < gap;
  if (!any) return;
  double* V = STAGED ? stage : Z;
  if (STAGED) {
    for (int x = tid; x < k * n; x += NT) stage[x] = Z[x];
    __syncthreads();
  }
  for (int t = 1; t < k; ++t) {
    int s0 = t;  // first member of the cluster of t
    while (s0 > 0 && fabs(lam[s0 - 1] - lam[t]) < gap) --s0;
    if (s0 == t) continue;
    double* vt = V + static_cast<long>(t) * n;
    for (int pass = 0; pass < 2; ++pass) {
      for (int s = s0 + wave; s < t; s += NT / 64) {
        const double* vs = V + static_cast<long>(s) * n;
        double dot = 0.0;
        for (int i = lane; i < n; i += 64) dot += vs[i] * vt[i];
        dot = wave_sum64(dot);
        if (lane == 0) red[s] = dot;
      }
      __syncthreads();
      if (tid < n) {
        double z = vt[tid];
        for (int s = s0; s < t; ++s) z -= red[s] * V[static_cast<long>(s) * n + tid];
        vt[tid] = z;
      }
      __syncthreads();
    }
    if (wave == 0) {
      double nr = 0.0;
      for (int i = lane; i < n; i += 64) nr += vt[i] * vt[i];
      nr = wave_sum64(nr);
      if (lane == 0) red[KMAX - 1] = 1.0 / sqrt(nr);
    }
    __syncthreads();
    if (tid < n) vt[tid] *= red[KMAX - 1];
    __syncthreads();
  }
  if (STAGED)
    for (int x = tid; x < k * n; x += NT) Z[x] = stage[x];
}

template <bool STAGED>
__global__ void __launch_bounds__(kClusterThreads) cluster_kernel(int n, int k, const double* __restrict__ lam,
                                                                  const double* __restrict__ norm, double* Z) {
  orthogonalise_clusters<STAGED, kClusterThreads, kClusterLds, 512>(n, k, lam, norm, Z);
}

// ---------------------------------------------------------------- 4. y = Q z

// Reflectors in reverse order, two at a time: with s1 = t1 v1.z and s2 =
// t2 (v2.z - s1 v2.v1) the sums of a pair are independent of each other, so
// a pair costs the latency of one.  The next four reflectors are loaded while
// four are applied.
template <int NC>
__device__ __forceinline__ void reflect(int tt, int n, int lda, const double* __restrict__ W,
                                        const double* __restrict__ tau, const double* __restrict__ Z,
                                        double* __restrict__ A) {
  const int lane = threadIdx.x & 63;
  double z[NC], tr[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int i = lane + 64 * c;
    z[c] = i < n ? Z[static_cast<long>(tt) * n + i] : 0.0;
    tr[c] = i < n ? tau[i] : 0.0;
  }
  double cur[4][NC], nxt[4][NC];
  auto load = [&](int j0, double (*v)[NC]) {  // reflectors j0, j0 - 1, ... (zero below 0)
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int j = j0 - u, i = lane + 64 * c;
        v[u][c] = (j >= 0 && i > j && i < n) ? W[static_cast<long>(j) * n + i] : 0.0;
      }
  };
  load(n - 3, cur);
  for (int j0 = n - 3; j0 >= 0; j0 -= 4) {
    load(j0 - 4, nxt);
#pragma unroll
    for (int u = 0; u < 4; u += 2) {
      const int j1 = j0 - u, j2 = j1 - 1;
      const double t1 = j1 >= 0 ? element<NC>(tr, max(j1, 0)) : 0.0, t2 = j2 >= 0 ? element<NC>(tr, max(j2, 0)) : 0.0;
      double d1 = 0.0, d2 = 0.0, d12 = 0.0;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        d1 += cur[u][c] * z[c];
        d2 += cur[u + 1][c] * z[c];
        d12 += cur[u][c] * cur[u + 1][c];
      }
      const double s1 = t1 * wave_sum64(d1);
      const double s2 = t2 * fma(-s1, wave_sum64(d12), wave_sum64(d2));
#pragma unroll
      for (int c = 0; c < NC; ++c) z[c] = fma(-s2, cur[u + 1][c], fma(-s1, cur[u][c], z[c]));
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int c = 0; c < NC; ++c) cur[u][c] = nxt[u][c];
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int i = lane + 64 * c;
    if (i < n) A[static_cast<long>(tt) * lda + i] = z[c];
  }
}

template <int NC>
__global__ void __launch_bounds__(64) reflect_kernel(int n, int lda, const double* __restrict__ W,
                                                     const double* __restrict__ tau,
                                                     const double* __restrict__ lam, const double* __restrict__ Z,
                                                     double* __restrict__ A, double* __restrict__ w,
                                                     const int* __restrict__ failed, int* __restrict__ info,
                                                     double* __restrict__ status) {
  const int tt = blockIdx.x, word = failed && *failed ? kEigGaveUp : 0;
  if (word == 0) {
    reflect<NC>(tt, n, lda, W, tau, Z, A);
    if (threadIdx.x == 0) w[tt] = lam[tt];
  }
  if (tt == 0 && threadIdx.x == 0) {
    info[0] = word;
    if (status) *status = word;
  }
}

// ---------------------------------------------------------------- many problems

// Scratch of one problem of a batch: reflectors, eigenvectors of T, (d, tau, e), eigenvalues and |T|.
struct BatchScratch {
  double *W, *Z, *dte, *lam, *norm;
  __device__ BatchScratch(const EigBatch& b, int m) {
    W = b.scratch + static_cast<long>(m) * b.scratch_stride;
    Z = W + b.ld * b.ld;
    dte = Z + b.kcap * b.ld;
    lam = dte + 3 * b.ld;
    norm = lam + b.kcap;
  }
};

__device__ __forceinline__ int batch_pairs(const EigBatch& b, int n) {
  return min(n, n + b.kfew > b.ld ? b.kcap : b.kfew);
}

__global__ void __launch_bounds__(512) batch_tridiag_kernel(EigBatch b) {
  const int m = blockIdx.x;
  if (!b.active[m]) return;
  const BatchScratch s(b, m);
  tridiagonalise<1, 8, 8, false>(b.n[m], b.A + static_cast<long>(m) * b.ld * b.ld, b.ld, s.W, s.dte, nullptr, nullptr, 0);
}

__global__ void __launch_bounds__(kPairThreads) batch_pair_kernel(EigBatch b) {
  const int m = blockIdx.x, t = blockIdx.y;
  if (!b.active[m] || t >= batch_pairs(b, b.n[m])) return;
  const BatchScratch s(b, m);
  tridiag_pair<1>(t, b.n[m], s.dte, s.lam, s.Z, s.norm);
}

// clusters, then y = Q z, one wavefront per vector
__global__ void __launch_bounds__(256) batch_vectors_kernel(EigBatch b) {
  const int m = blockIdx.x;
  if (!b.active[m]) return;
  const BatchScratch s(b, m);
  const int n = b.n[m], k = batch_pairs(b, n);
  orthogonalise_clusters<true, 256, kEigBatchPairs * 64, kEigBatchPairs + 1>(n, k, s.lam, s.norm, s.Z);
  __syncthreads();  // orders the workgroup's own stores to Z
  double* out = b.vec + static_cast<long>(m) * b.ld * b.ld;
  for (int t = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); t < k; t += 4)
    reflect<1>(t, n, b.ld, s.W, s.dte + 2 * n, s.Z, out);
  for (int t = threadIdx.x; t < k; t += 256) b.val[static_cast<long>(m) * b.ld + t] = s.lam[t];
}

// scratch layout (doubles)
struct EigScratch {
  double *W, *Z, *dte, *lam, *norm, *failed, *xch;
  EigScratch(double* s, int n, int k) {
    W = s;
    Z = W + static_cast<long>(n) * n;
    dte = Z + static_cast<long>(n) * k;
    lam = dte + 3 * n;
    norm = lam + k;
    failed = norm + 1;
    xch = failed + 1;
  }
};

template <int NC>
void launch_tail(hipStream_t st, int n, double* A, int lda, int k, double* w, const EigScratch& s, const int* failed,
                 int* info, double* status) {
  hipLaunchKernelGGL(tridiag_pair_kernel<NC>, dim3(k), dim3(kPairThreads), 0, st, n, s.dte, s.lam, s.Z, s.norm);
  if (k > 1) {
    if (static_cast<long>(k) * n <= kClusterLds)
      hipLaunchKernelGGL(cluster_kernel<true>, dim3(1), dim3(kClusterThreads), 0, st, n, k, s.lam, s.norm, s.Z);
    else
      hipLaunchKernelGGL(cluster_kernel<false>, dim3(1), dim3(kClusterThreads), 0, st, n, k, s.lam, s.norm, s.Z);
  }
  hipLaunchKernelGGL(reflect_kernel<NC>, dim3(k), dim3(64), 0, st, n, lda, s.W, s.dte + 2 * n, s.lam, s.Z, A, w,
                     failed, info, status);
}

template <int NC, int NR, int NW, bool GRID>
void launch_tridiag(hipStream_t st, int n, const double* A, int lda, const EigScratch& s, int poll_limit) {
  int* failed = reinterpret_cast<int*>(s.failed);
  if constexpr (GRID) {
    const long nx = 2L * n * n;
    hipLaunchKernelGGL(exchange_fill_kernel, dim3(ceil_div(nx, 256)), dim3(256), 0, st, nx,
                       reinterpret_cast<unsigned long long*>(s.xch), failed);
    hipLaunchKernelGGL((tridiag_kernel<NC, NR, NW, true>), dim3(NW), dim3(64), 0, st, n, A, lda, s.W, s.dte, s.xch,
                       failed, poll_limit);
  } else {
    hipLaunchKernelGGL((tridiag_kernel<NC, NR, NW, false>), dim3(1), dim3(64 * NW), 0, st, n, A, lda, s.W, s.dte,
                       s.xch, failed, 0);
  }
}

}  // namespace

size_t eig_batch_scratch(int ld, int kcap) {
  return static_cast<size_t>(ld) * ld + static_cast<size_t>(kcap) * ld + 3 * static_cast<size_t>(ld) + kcap + 1;
}

void launch_eig_batch(hipStream_t st, int nprob, const EigBatch& b) {
  if (b.ld > 64 || b.kcap > kEigBatchPairs || b.kfew > b.kcap ||
      static_cast<size_t>(b.scratch_stride) < eig_batch_scratch(b.ld, b.kcap))
    throw Error(kEArg, "eigenproblem batch out of range");
  hipLaunchKernelGGL(batch_tridiag_kernel, dim3(nprob), dim3(512), 0, st, b);
  hipLaunchKernelGGL(batch_pair_kernel, dim3(nprob, b.kcap), dim3(kPairThreads), 0, st, b);
  hipLaunchKernelGGL(batch_vectors_kernel, dim3(nprob), dim3(256), 0, st, b);
  SEQX_LAUNCH_CHECK();
}

size_t eig_lowest_scratch(int n, int k) {
  return static_cast<size_t>(n) * n + static_cast<size_t>(n) * k + 3 * static_cast<size_t>(n) + k + 2 +
         (n > kEigOneGroup ? 2 * static_cast<size_t>(n) * n : 0);
}

void launch_eig_lowest(hipStream_t st, int n, double* A, int lda, int k, double* w, double* scratch, int* info,
                       double* status, int poll_limit) {
  const EigScratch s(scratch, n, k);
  if (n <= 64) launch_tridiag<1, 8, 8, false>(st, n, A, lda, s, poll_limit);
  else if (n <= 128) launch_tridiag<2, 16, 8, false>(st, n, A, lda, s, poll_limit);
  else if (n <= 192) launch_tridiag<3, 8, 24, true>(st, n, A, lda, s, poll_limit);
  else if (n <= 256) launch_tridiag<4, 8, 32, true>(st, n, A, lda, s, poll_limit);
  else if (n <= 384) launch_tridiag<6, 8, 48, true>(st, n, A, lda, s, poll_limit);
  else launch_tridiag<8, 8, 64, true>(st, n, A, lda, s, poll_limit);
  const int* failed = n > kEigOneGroup ? reinterpret_cast<const int*>(s.failed) : nullptr;
  if (n <= 64) launch_tail<1>(st, n, A, lda, k, w, s, failed, info, status);
  else if (n <= 128) launch_tail<2>(st, n, A, lda, k, w, s, failed, info, status);
  else if (n <= 256) launch_tail<4>(st, n, A, lda, k, w, s, failed, info, status);
  else launch_tail<8>(st, n, A, lda, k, w, s, failed, info, status);
  SEQX_LAUNCH_CHECK();
}

}  // namespace seqx
