// Batched CIS Davidson (batched outline of the paper's GPU-implementation
// subsection and its Fig. 2) for many small molecules of uneven size.
//
// The paper pads every molecule to the largest and runs dense batched tensor
// operations.  Here nothing is padded: a (molecule, trial vector) pair is a
// work item, and one persistent launch of a fused kernel forms all products of
// an iteration.  Each 256-thread workgroup takes items in a static round-robin
// over a list ordered by molecule size (largest first), and for one item runs
// Eqs. 8-9 end to end:
//   T = C_o V,  R = T C_v^T           (workgroup MFMA GEMMs)
//   F = 2 J(R) - K(R)                 (packed Coulomb, one-centre and pair exchange)
//   Z = F C_v,  A V = C_o^T Z + de V  (workgroup MFMA GEMMs, FP64 epilogue)
// with R, F and T/Z in a per-workgroup slice of global scratch (L2-resident).
// The subspace steps (projection, eigensolve, Ritz vectors and
// residuals, preconditioning, collapse, Gram-Schmidt) are one launch each over
// all molecules, with per-molecule flags on the device, so the iteration is a
// fixed sequence of launches (captured once as a HIP graph); the host reads one
// counter per iteration.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <type_traits>

#include "batch.hpp"
#include "wave.hpp"
#include "fock_blocks.hpp"
#include "linalg.hpp"

namespace seqx {

static_assert(kBatchMaxSub <= 64 && 2 * kBatchMaxRoots <= kEigBatchPairs, "range of the batched eigensolver");

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef double d4 __attribute__((ext_vector_type(4)));

template <class T>
struct WgMfma;
template <>
struct WgMfma<float> {
  typedef f4 acc_t;
  static __device__ __forceinline__ acc_t op(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};
template <>
struct WgMfma<double> {
  typedef d4 acc_t;
  static __device__ __forceinline__ acc_t op(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};

// Workgroup GEMM (4 wavefronts): out(i, j) = sum_k A(i, k) B(k, j) for i < M,
// j < N, with A(i, k) = A[i sai + k sak] and B(k, j) = B[k sbk + j sbj] (any
// transposition through the strides).  Each wave owns macro tiles of
// (16 TM) x (16 TN) in round-robin; operands come straight from global memory
// (L1/L2) in the MFMA lane layout; store(i, j, value) writes the result.
template <class T, int TM, int TN, class TA, class TB, class Store>
__device__ __forceinline__ void wg_gemm(int M, int N, int K, const TA* __restrict__ A, long sai, long sak,
                                        const TB* __restrict__ B, long sbk, long sbj, Store store) {
  typedef WgMfma<T> MF;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r16 = lane & 15, k4 = lane >> 4;
  const int tm = (M + 16 * TM - 1) / (16 * TM), tn = (N + 16 * TN - 1) / (16 * TN);
  const int nwave = blockDim.x >> 6;
  for (int t = wave; t < tm * tn; t += nwave) {
    const int i0 = (t / tn) * 16 * TM, j0 = (t % tn) * 16 * TN;
    typename MF::acc_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = typename MF::acc_t{0, 0, 0, 0};
    // four k-steps per pass, all loads first (the loads past K read zero, so
    // no remainder loop is needed)
    for (int k0 = 0; k0 < K; k0 += 16) {
      T a[4][TM], b[4][TN];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = k0 + 4 * q + k4;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int row = i0 + i * 16 + r16;
          a[q][i] = (row < M && k < K) ? static_cast<T>(A[row * sai + k * sak]) : T(0);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int col = j0 + j * 16 + r16;
          b[q][j] = (col < N && k < K) ? static_cast<T>(B[k * sbk + col * sbj]) : T(0);
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = MF::op(a[q][i], b[q][j], acc[i][j]);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = i0 + i * 16 + MF::row(lane, r), col = j0 + j * 16 + r16;
          if (row < M && col < N) store(row, col, static_cast<double>(acc[i][j][r]));
        }
  }
}

constexpr int kSigThreads = 256;  // threads per work item (512 measured slower: the phases are latency-bound)

// One CIS product A V for one trial vector of one molecule (whole workgroup).
// scr: n*n (R) + n*n (F) + n*v (T, then Z) elements of T; rs, js: LDS [np].
template <class T, int TM, int TN>
__device__ void sigma_item(const MolDesc& md, const T* __restrict__ C, const double* __restrict__ V,
                           double* __restrict__ out, T* __restrict__ scr, double* rs, double* js) {
  const int n = md.n, o = md.o, v = md.v, np = md.np;
  T* R = scr;
  T* F = scr + static_cast<long>(n) * n;
  T* Tz = scr + 2L * n * n;
  // T (n x v) = C[:, :o] V
  wg_gemm<T, TM, TN>(n, v, o, C, n, 1, V, v, 1,
                     [&](int i, int j, double x) { Tz[static_cast<long>(i) * v + j] = static_cast<T>(x); });
  __syncthreads();
  // R (n x n) = T C[:, o:]^T
  wg_gemm<T, TM, TN>(n, n, v, Tz, v, 1, C + o, 1, n,
                     [&](int i, int j, double x) { R[static_cast<long>(i) * n + j] = static_cast<T>(x); });
  __syncthreads();
  // packed same-atom densities r_P and Coulomb J = W r (one wave per row, fixed-order reduction)
  for (int P = threadIdx.x; P < np; P += blockDim.x) {
    const int mu = md.pi_mu[P], nu = md.pi_nu[P];
    const double a = static_cast<double>(R[static_cast<long>(mu) * n + nu]);
    const double b = static_cast<double>(R[static_cast<long>(nu) * n + mu]);
    rs[P] = (mu == nu) ? a : a + b;
  }
  __syncthreads();
  // J[P] = sum_Q W[Q][P] r[Q] (W symmetric): thread P walks column P, so each
  // step reads one row of W coalesced and no cross-lane sum is needed
  for (int P0 = 0; P0 < np; P0 += blockDim.x) {
    const int P = P0 + threadIdx.x;
    const double* Wc = md.W + min(P, np - 1);
    double s0 = 0.0, s1 = 0.0;
    int Q = 0;
    for (; Q + 2 <= np; Q += 2) {
      s0 += Wc[static_cast<long>(Q) * np] * rs[Q];
      s1 += Wc[static_cast<long>(Q + 1) * np] * rs[Q + 1];
    }
    if (Q < np) s0 += Wc[static_cast<long>(Q) * np] * rs[Q];
    if (P < np) js[P] = s0 + s1;
  }
  __syncthreads();
  // F = 2 J(R) - K(R): atom-diagonal blocks, then every atom pair (both orders)
  for (int A = threadIdx.x; A < md.natoms; A += blockDim.x)
    diag_block<kSum, T>(md.elems[md.slot[A]], md.ao_off[A], md.pi_off[A], js, 1, R, n, MatOut<T>{F, 0, n},
                        MatOut<T>{nullptr, 0, n}, 2.0, -1.0, -1.0);
  for (int p = threadIdx.x; p < md.npairs[0]; p += blockDim.x)
    exchange_pair<4, 4, kSum, T, T>(md.pairs[0][p].x, md.pairs[0][p].y, md.ao_off, md.pi_off, md.W, np, R, n, F,
                                    static_cast<T*>(nullptr), -1.0, -1.0);
  for (int p = threadIdx.x; p < md.npairs[1]; p += blockDim.x)
    exchange_pair<4, 1, kSum, T, T>(md.pairs[1][p].x, md.pairs[1][p].y, md.ao_off, md.pi_off, md.W, np, R, n, F,
                                    static_cast<T*>(nullptr), -1.0, -1.0);
  for (int p = threadIdx.x; p < md.npairs[2]; p += blockDim.x)
    exchange_pair<1, 1, kSum, T, T>(md.pairs[2][p].x, md.pairs[2][p].y, md.ao_off, md.pi_off, md.W, np, R, n, F,
                                    static_cast<T*>(nullptr), -1.0, -1.0);
  __syncthreads();
  // Z (n x v) = F C[:, o:]
  wg_gemm<T, TM, TN>(n, v, n, F, n, 1, C + o, n, 1,
                     [&](int i, int j, double x) { Tz[static_cast<long>(i) * v + j] = static_cast<T>(x); });
  __syncthreads();
  // A V (o x v) = C[:, :o]^T Z + (eps_a - eps_i) V, the diagonal term in FP64
  const double* eps = md.eps;
  wg_gemm<T, TM, TN>(o, v, n, C, 1, n, Tz, v, 1, [&](int i, int j, double x) {
    const long ij = static_cast<long>(i) * v + j;
    out[ij] = x + (eps[o + j] - eps[i]) * V[ij];
  });
  __syncthreads();
}

// counters: [0] number of items, [1] active molecules, [2] iteration
template <class T>
__global__ void __launch_bounds__(kSigThreads) sigma_items_kernel(const MolDesc* __restrict__ mols,
                                                          const int2* __restrict__ items, const int* __restrict__ counters,
                                                          const double* __restrict__ Vp, double* __restrict__ AVp,
                                                          T* __restrict__ scratch, long scratch_stride,
                                                          long long* __restrict__ stamps) {
  __shared__ double rs[kBatchMaxNp];
  __shared__ double js[kBatchMaxNp];
  if (threadIdx.x == 0) stamps[2 * blockIdx.x] = static_cast<long long>(wall_clock64());
  const int nit = counters[0];
  T* scr = scratch + blockIdx.x * scratch_stride;
  for (int it = blockIdx.x; it < nit; it += gridDim.x) {
    const int2 item = items[it];
    const MolDesc md = mols[item.x];
    const T* C = sizeof(T) == 4 ? reinterpret_cast<const T*>(md.C32) : reinterpret_cast<const T*>(md.C64);
    const double* V = Vp + md.vbase + item.y * md.nov;
    double* out = AVp + md.vbase + item.y * md.nov;
    switch (md.variant) {
      case 0: sigma_item<T, 1, 1>(md, C, V, out, scr, rs, js); break;
      case 1: sigma_item<T, 2, 1>(md, C, V, out, scr, rs, js); break;
      default: sigma_item<T, 2, 2>(md, C, V, out, scr, rs, js); break;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) stamps[2 * blockIdx.x + 1] = static_cast<long long>(wall_clock64());
}

// Span of the last sigma launch (latest end - earliest start over its
// workgroups, device wall-clock ticks), added to acc[0]; fixed-order reduction.
__global__ void __launch_bounds__(256) stamp_span_kernel(int G, const long long* __restrict__ stamps,
                                                         long long* acc) {
  __shared__ long long lo[256], hi[256];
  long long a = 0x7fffffffffffffffLL, b = 0;
  for (int i = threadIdx.x; i < G; i += 256) {
    a = min(a, stamps[2 * i]);
    b = max(b, stamps[2 * i + 1]);
  }
  lo[threadIdx.x] = a;
  hi[threadIdx.x] = b;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h) {
      lo[threadIdx.x] = min(lo[threadIdx.x], lo[threadIdx.x + h]);
      hi[threadIdx.x] = max(hi[threadIdx.x], hi[threadIdx.x + h]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) acc[0] += hi[0] - lo[0];
}

// ---------------------------------------------------------------- subspace kernels

__device__ __forceinline__ double wave_sum(double s) { return wave_sum64(s); }

// fixed-order block sum over 256 threads (result valid in every thread)
__device__ double block_sum(double s, double* red) {  // 256 threads; fixed order
  s = wave_sum64(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  const double r = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return r;
}

// Gap guess: unit vectors at the ng = min(nov, 2K) smallest eps_a - eps_i
// (ties by flat index i*v + a), found by ng rounds of lexicographic minimum.
__global__ void __launch_bounds__(256) guess_kernel(int nmol, const MolDesc* __restrict__ mols, int K,
                                                    double* __restrict__ Vp, int* S, int* knew, int* active, int* conv,
                                                    int* coll, int* qcol) {
  __shared__ double bg[256];
  __shared__ long bi[256];
  const int m = blockIdx.x;
  const MolDesc md = mols[m];
  const long nov = md.nov;
  const int ng = static_cast<int>(nov < 2L * K ? nov : 2L * K);
  double* V = Vp + md.vbase;
  for (long x = threadIdx.x; x < ng * nov; x += 256) V[x] = 0.0;
  __syncthreads();
  double lg = -1e300;
  long li = -1;
  for (int r = 0; r < ng; ++r) {
    double g = 1e300;
    long gi = nov;
    for (long x = threadIdx.x; x < nov; x += 256) {
      const double d = md.eps[md.o + x % md.v] - md.eps[x / md.v];
      const bool after = d > lg || (d == lg && x > li);
      if (after && (d < g || (d == g && x < gi))) {
        g = d;
        gi = x;
      }
    }
    bg[threadIdx.x] = g;
    bi[threadIdx.x] = gi;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
      if (threadIdx.x < h) {
        const double g2 = bg[threadIdx.x + h];
        const long i2 = bi[threadIdx.x + h];
        if (g2 < bg[threadIdx.x] || (g2 == bg[threadIdx.x] && i2 < bi[threadIdx.x])) {
          bg[threadIdx.x] = g2;
          bi[threadIdx.x] = i2;
        }
      }
      __syncthreads();
    }
    lg = bg[0];
    li = bi[0];
    if (threadIdx.x == 0) V[r * nov + li] = 1.0;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    S[m] = 0;
    knew[m] = ng;
    active[m] = 1;
    conv[m] = 0;
    coll[m] = 0;
    qcol[m] = 0;
  }
}

// Work list of the iteration: items (m, S_m + j), j < knew_m, molecules in
// the size order `order` (largest first); block-wide exclusive scan.
__global__ void __launch_bounds__(256) items_kernel(int nmol, const MolDesc* __restrict__ mols,
                                                    const int* __restrict__ order, const int* __restrict__ S,
                                                    const int* __restrict__ knew, const int* __restrict__ active,
                                                    int2* __restrict__ items, int* counters, long long* nsig) {
  __shared__ int part[256];
  __shared__ long long fl[256];
  const int per = (nmol + 255) / 256;
  const int b0 = threadIdx.x * per, b1 = min(nmol, b0 + per);
  int cnt = 0;
  long long flops = 0;  // algorithmic transform flops of the items: 4 n v (n + o) each
  for (int q = b0; q < b1; ++q) {
    const int m = order[q];
    if (active[m]) {
      cnt += knew[m];
      const long long n = mols[m].n, o = mols[m].o, v = mols[m].v;
      flops += knew[m] * 4LL * n * v * (n + o);
    }
  }
  part[threadIdx.x] = cnt;
  fl[threadIdx.x] = flops;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h) fl[threadIdx.x] += fl[threadIdx.x + h];
    __syncthreads();
  }
  for (int h = 1; h < 256; h <<= 1) {  // inclusive Hillis-Steele scan
    const int add = threadIdx.x >= h ? part[threadIdx.x - h] : 0;
    __syncthreads();
    part[threadIdx.x] += add;
    __syncthreads();
  }
  int pos = part[threadIdx.x] - cnt;
  for (int q = b0; q < b1; ++q) {
    const int m = order[q];
    if (!active[m]) continue;
    for (int j = 0; j < knew[m]; ++j) items[pos++] = make_int2(m, S[m] + j);
  }
  if (threadIdx.x == 255) {
    counters[0] = part[255];
    nsig[0] += part[255];
    nsig[2] += fl[0];
  }
}

// Subspace steps of a molecule are split over blocks along its nov entries, so
// that the largest molecules spread over several CUs: chunks of about 256
// entries (one a thread in the row combinations), at most kXChunks.  Partial
// inner products go to per-chunk slots and are summed in a fixed order.
constexpr int kXChunks = 8;
constexpr int kPartStride = kBatchMaxSub * 2 * kBatchMaxRoots;  // one chunk's [s][j] partials

__device__ __forceinline__ int chunks_of(long nov) {
  return static_cast<int>(min(static_cast<long>(kXChunks), (nov + 255) / 256));
}
__device__ __forceinline__ long chunk_begin(long nov, int ch) {
  const int nch = chunks_of(nov);
  const long len = ((nov + nch - 1) / nch + 15) / 16 * 16;
  return min(nov, len * ch);
}

struct __attribute__((packed, aligned(8))) Row4 {  // four row elements at any element offset
  double v[4];
};

constexpr int kSubTiles = (kBatchMaxSub + 15) / 16;
struct DotsLds {
  double part[4][kSubTiles][16][17];
};

// P[s * 2 kBatchMaxRoots + u] = sum over x in [x0, x1) of V_s[x] b_u[x] for s <
// ns, u < nb <= 16, one workgroup of 4 wavefronts.  b is this lane's column
// (that of u = lane & 15, any valid row for u >= nb).  The products are 16 x 16
// tiles of the FP64 matrix cores, so nothing is summed across lanes and every
// element of V is read once; a lane takes four neighbouring elements of its row
// and the k index of the tile is permuted alike on both sides.  (One wavefront
// per two rows with a lane sum for each product: 325 us for the two passes of a
// Gram-Schmidt step over 512 molecules with 20 rows, here 89.)
__device__ __forceinline__ void chunk_dots(const double* __restrict__ V, long nov, int ns,
                                           const double* __restrict__ b, int nb, long x0, long x1,
                                           double* __restrict__ P, DotsLds& L) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, k4 = lane >> 4, nt = (ns + 15) / 16;
  const long len = (x1 - x0 + 63) / 64 * 16, xa = x0 + wave * len, xb = min(x1, xa + len);
  const double* row[kSubTiles];
  d4 acc[kSubTiles];
#pragma unroll
  for (int t = 0; t < kSubTiles; ++t) {
    row[t] = V + static_cast<long>(min(16 * t + r16, ns - 1)) * nov;
    acc[t] = d4{0, 0, 0, 0};
  }
  for (long x = xa; x < xb; x += 16) {
    const long xl = x + 4 * k4;
    Row4 bv, av[kSubTiles];
    if (x + 16 <= xb) {
      bv = *reinterpret_cast<const Row4*>(b + xl);
#pragma unroll
      for (int t = 0; t < kSubTiles; ++t)
        if (t < nt) av[t] = *reinterpret_cast<const Row4*>(row[t] + xl);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        bv.v[i] = xl + i < xb ? b[xl + i] : 0.0;
#pragma unroll
        for (int t = 0; t < kSubTiles; ++t)
          if (t < nt) av[t].v[i] = xl + i < xb ? row[t][xl + i] : 0.0;
      }
    }
#pragma unroll
    for (int t = 0; t < kSubTiles; ++t)
      if (t < nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[t] = WgMfma<double>::op(av[t].v[i], bv.v[i], acc[t]);
  }
  __syncthreads();  // L may still be read from the previous call
#pragma unroll
  for (int t = 0; t < kSubTiles; ++t)
    if (t < nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) L.part[wave][t][WgMfma<double>::row(lane, r)][r16] = acc[t][r];
  __syncthreads();
  for (int idx = threadIdx.x; idx < 16 * ns; idx += 256) {
    const int sidx = idx >> 4, u = idx & 15, t = sidx >> 4, i = sidx & 15;
    if (u < nb)
      P[sidx * 2 * kBatchMaxRoots + u] =
          (L.part[0][t][i][u] + L.part[1][t][i][u]) + (L.part[2][t][i][u] + L.part[3][t][i][u]);
  }
}

// acc[j] = sum_s c[s][j] row_s[x] over n rows (ld nov), four rows' loads ahead
// of their products; c is zero-padded to a multiple of four rows
template <int NR>
__device__ __forceinline__ void combine_at(const double* __restrict__ rows, long nov, int n, long x,
                                           const double (*c)[NR], double (&acc)[NR]) {
  for (int s0 = 0; s0 < n; s0 += 4) {
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = rows[min(s0 + q, n - 1) * nov + x];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int j = 0; j < NR; ++j) acc[j] += c[s0 + q][j] * v[q];
  }
}

// New columns of M = V^T A V, first half: block (m, c) forms the partial
// inner products over chunk c of every new product A V_j (j < knew_m, in
// groups of 16) with every basis row s < S_m + knew_m.
__global__ void __launch_bounds__(256) project_part_kernel(const MolDesc* __restrict__ mols,
                                                           const double* __restrict__ Vp,
                                                           const double* __restrict__ AVp, const int* __restrict__ S,
                                                           const int* __restrict__ knew,
                                                           const int* __restrict__ active, double* __restrict__ part) {
  __shared__ DotsLds L;
  const int m = blockIdx.x, ch = blockIdx.y;
  if (!active[m]) return;
  const MolDesc md = mols[m];
  const long nov = md.nov;
  if (ch >= chunks_of(nov)) return;
  const int S0 = S[m], kn = knew[m];
  double* P = part + (static_cast<long>(m) * kXChunks + ch) * kPartStride;
  for (int j0 = 0; j0 < kn; j0 += 16) {
    const int nb = min(16, kn - j0);
    const double* b = AVp + md.vbase + static_cast<long>(S0 + j0 + min(static_cast<int>(threadIdx.x & 15), nb - 1)) * nov;
    chunk_dots(Vp + md.vbase, nov, S0 + kn, b, nb, chunk_begin(nov, ch), chunk_begin(nov, ch + 1), P + j0, L);
  }
}

// Second half: sum the chunks in order and write both triangles of the new
// columns (column-major, ld Smax).  S is advanced by advance_kernel afterwards.
__global__ void __launch_bounds__(256) project_kernel(const MolDesc* __restrict__ mols, int Smax,
                                                      const double* __restrict__ part,
                                                      double* __restrict__ Mp, const int* __restrict__ S,
                                                      const int* __restrict__ knew, const int* __restrict__ active) {
  const int m = blockIdx.x;
  if (!active[m]) return;
  const int S0 = S[m], kn = knew[m], ns = S0 + kn;
  double* M = Mp + static_cast<long>(m) * Smax * Smax;
  const double* P = part + static_cast<long>(m) * kXChunks * kPartStride;
  const int nch = chunks_of(mols[m].nov);
  for (int idx = threadIdx.x; idx < ns * kn; idx += 256) {
    const int sidx = idx / kn, jn = idx % kn, j = S0 + jn;
    if (sidx > j) continue;
    double d = 0.0;
    for (int c = 0; c < nch; ++c) d += P[c * kPartStride + sidx * 2 * kBatchMaxRoots + jn];
    M[sidx + static_cast<long>(j) * Smax] = d;
    M[j + static_cast<long>(sidx) * Smax] = d;
  }
}

__global__ void advance_kernel(int nmol, int* S, const int* __restrict__ knew, const int* __restrict__ active) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m < nmol && active[m]) S[m] += knew[m];
}

// Ritz vectors of molecule m, X_j = sum_s evec(s, j) V_s, and residuals
// r_j = A X_j - w_j X_j into Wc, for all K <= NR roots in one pass over V and A V
// (each basis element read once); block (m, c) takes chunk c of the nov
// entries and leaves its partial sums of |r_j|^2 in rpart[m][c][j].
template <int NR>
__global__ void __launch_bounds__(256) ritz_kernel(const MolDesc* __restrict__ mols, int K, int Smax,
                                                   const double* __restrict__ Vp, const double* __restrict__ AVp,
                                                   const double* __restrict__ evec, const double* __restrict__ eval,
                                                   const int* __restrict__ S, const int* __restrict__ active,
                                                   double* __restrict__ Xp, double* __restrict__ Wcp,
                                                   double* __restrict__ omega, double* __restrict__ rpart) {
  __shared__ double c[kBatchMaxSub][NR];
  __shared__ double wr[NR];
  __shared__ double red[4][NR];
  const int m = blockIdx.x, ch = blockIdx.y;
  if (!active[m]) return;
  const MolDesc md = mols[m];
  const long nov = md.nov;
  if (ch >= chunks_of(nov)) return;
  const int n = S[m];
  for (int idx = threadIdx.x; idx < kBatchMaxSub * NR; idx += 256) {
    const int sidx = idx / NR, j = idx % NR;
    c[sidx][j] = (sidx < n && j < K) ? evec[static_cast<long>(m) * Smax * Smax + sidx + static_cast<long>(j) * Smax] : 0.0;
  }
  if (threadIdx.x < NR) wr[threadIdx.x] = threadIdx.x < K ? eval[static_cast<long>(m) * Smax + threadIdx.x] : 0.0;
  __syncthreads();
  double* X = Xp + md.xbase;
  double* Wc = Wcp + md.xbase;
  const long x0 = chunk_begin(nov, ch), x1 = chunk_begin(nov, ch + 1);
  double ss[NR];
#pragma unroll
  for (int j = 0; j < NR; ++j) ss[j] = 0.0;
  for (long x = x0 + threadIdx.x; x < x1; x += 256) {
    double xv[NR] = {}, av[NR] = {};
    combine_at<NR>(Vp + md.vbase, nov, n, x, c, xv);
    combine_at<NR>(AVp + md.vbase, nov, n, x, c, av);
#pragma unroll
    for (int j = 0; j < NR; ++j)
      if (j < K) {
        const double r = av[j] - wr[j] * xv[j];
        X[j * nov + x] = xv[j];
        Wc[j * nov + x] = r;
        ss[j] += r * r;
      }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < NR; ++j)
    if (j < K) {
      const double t = wave_sum(ss[j]);
      if (lane == 0) red[wave][j] = t;
    }
  __syncthreads();
  if (threadIdx.x < K)
    rpart[(static_cast<long>(m) * kXChunks + ch) * kBatchMaxRoots + threadIdx.x] =
        (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
  if (ch == 0 && threadIdx.x < K) omega[m * K + threadIdx.x] = wr[threadIdx.x];
}

// Convergence and bookkeeping for every molecule; counts the active ones.
__global__ void __launch_bounds__(256) select_kernel(int nmol, const MolDesc* __restrict__ mols, int K, int Smax,
                                                     double tol,
                                                     const double* __restrict__ rpart, double* __restrict__ rnorm,
                                                     const int* __restrict__ S, int* knew, int* active, int* coll,
                                                     int* qcol, int* unc, int* conv, int* counters) {
  __shared__ double red[256];
  const int iter = counters[2] + 1;
  double nact = 0.0;
  for (int m = threadIdx.x; m < nmol; m += 256) {
    if (!active[m]) continue;
    int nu = 0;
    const int nch = chunks_of(mols[m].nov);
    for (int j = 0; j < K; ++j) {
      double r2 = 0.0;
      for (int c = 0; c < nch; ++c) r2 += rpart[(static_cast<long>(m) * kXChunks + c) * kBatchMaxRoots + j];
      const double rn = sqrt(r2);
      rnorm[m * K + j] = rn;
      if (rn > tol) unc[m * K + nu++] = j;
    }
    if (nu == 0) {
      active[m] = 0;
      conv[m] = iter;
      continue;
    }
    knew[m] = nu;
    coll[m] = S[m] + nu > Smax ? 1 : 0;
    qcol[m] = min(2 * K, S[m]);
    nact += 1.0;
  }
  nact = block_sum(nact, red);
  if (threadIdx.x == 0) {
    counters[1] = static_cast<int>(nact);
    counters[2] = iter;
  }
}

// Collapse onto the q <= NQ lowest Ritz vectors, V_s <- sum_t evec(t, s) V_t (and
// A V), in place: a thread forms all q new elements of its entry before it
// writes them.  The projected matrix becomes diag(lowest q eigenvalues).
template <int NQ>
__global__ void __launch_bounds__(256) collapse_kernel(const MolDesc* __restrict__ mols, int Smax,
                                                       double* __restrict__ Vp, double* __restrict__ AVp,
                                                       const double* __restrict__ evec,
                                                       const double* __restrict__ eval, const int* __restrict__ S,
                                                       const int* __restrict__ coll, const int* __restrict__ qcol,
                                                       double* __restrict__ Mp) {
  __shared__ double c[kBatchMaxSub][NQ];
  const int m = blockIdx.x, ch = blockIdx.y;
  if (!coll[m]) return;
  const MolDesc md = mols[m];
  const long nov = md.nov;
  if (ch >= chunks_of(nov)) return;
  const int n = S[m], q = qcol[m];
  for (int idx = threadIdx.x; idx < kBatchMaxSub * NQ; idx += 256) {
    const int t = idx / NQ, j = idx % NQ;
    c[t][j] = (t < n && j < q) ? evec[static_cast<long>(m) * Smax * Smax + t + static_cast<long>(j) * Smax] : 0.0;
  }
  __syncthreads();
  const long x0 = chunk_begin(nov, ch), x1 = chunk_begin(nov, ch + 1);
  for (long x = x0 + threadIdx.x; x < x1; x += 256)
    for (double* rows : {Vp + md.vbase, AVp + md.vbase}) {
      double acc[NQ] = {};
      combine_at<NQ>(rows, nov, n, x, c, acc);
#pragma unroll
      for (int j = 0; j < NQ; ++j)
        if (j < q) rows[j * nov + x] = acc[j];
    }
  if (ch == 0) {
    double* M = Mp + static_cast<long>(m) * Smax * Smax;
    for (int idx = threadIdx.x; idx < q * q; idx += 256) {
      const int i = idx / q, j = idx % q;
      M[i + static_cast<long>(j) * Smax] = (i == j) ? eval[static_cast<long>(m) * Smax + i] : 0.0;
    }
  }
}

// Corrections of the unconverged roots, first step: precondition the
// residuals in place, r / (w - de) with |w - de| kept >= 1e-8, and leave the
// partial sums of their squared norms per chunk (the norms before deflation).
__global__ void __launch_bounds__(256) precond_kernel(const MolDesc* __restrict__ mols, int K,
                                                      double* __restrict__ Wcp, const int* __restrict__ knew,
                                                      const int* __restrict__ active, const int* __restrict__ unc,
                                                      const double* __restrict__ omega, double* __restrict__ n0part) {
  __shared__ double wu[kBatchMaxRoots];
  __shared__ double red[4][kBatchMaxRoots];
  const int m = blockIdx.x, ch = blockIdx.y;
  if (!active[m]) return;
  const MolDesc md = mols[m];
  const long nov = md.nov, x0 = chunk_begin(nov, ch), x1 = chunk_begin(nov, ch + 1);
  if (ch >= chunks_of(nov)) return;
  const int nu = knew[m];
  double* w[kBatchMaxRoots];
#pragma unroll
  for (int u = 0; u < kBatchMaxRoots; ++u) w[u] = Wcp + md.xbase + unc[m * K + min(u, nu - 1)] * nov;
  if (threadIdx.x < nu) wu[threadIdx.x] = omega[m * K + unc[m * K + threadIdx.x]];
  __syncthreads();
  double n0[kBatchMaxRoots];
#pragma unroll
  for (int u = 0; u < kBatchMaxRoots; ++u) n0[u] = 0.0;
  for (long x = x0 + threadIdx.x; x < x1; x += 256) {
    const double de = md.eps[md.o + x % md.v] - md.eps[x / md.v];
#pragma unroll
    for (int u = 0; u < kBatchMaxRoots; ++u)
      if (u < nu) {
        double den = wu[u] - de;
        if (fabs(den) < 1e-8) den = den < 0.0 ? -1e-8 : 1e-8;
        const double t = w[u][x] / den;
        w[u][x] = t;
        n0[u] += t * t;
      }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int u = 0; u < kBatchMaxRoots; ++u)
    if (u < nu) {
      const double t = wave_sum(n0[u]);
      if (lane == 0) red[wave][u] = t;
    }
  __syncthreads();
  if (threadIdx.x < nu)
    n0part[(static_cast<long>(m) * kXChunks + ch) * kBatchMaxRoots + threadIdx.x] =
        (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
}

// Classical Gram-Schmidt of the corrections against the basis (its first
// qcol rows after a collapse), one half-pass each: partial inner products
// per chunk ...
__global__ void __launch_bounds__(256) gs_dots_kernel(const MolDesc* __restrict__ mols, int K,
                                                      const double* __restrict__ Vp, const double* __restrict__ Wcp,
                                                      const int* __restrict__ S, const int* __restrict__ knew,
                                                      const int* __restrict__ active, const int* __restrict__ coll,
                                                      const int* __restrict__ qcol, const int* __restrict__ unc,
                                                      double* __restrict__ part) {
  __shared__ DotsLds L;
  const int m = blockIdx.x, ch = blockIdx.y;
  if (!active[m]) return;
  const MolDesc md = mols[m];
  const long nov = md.nov;
  if (ch >= chunks_of(nov)) return;
  const int nb = coll[m] ? qcol[m] : S[m];
  const int nu = knew[m];
  const double* w = Wcp + md.xbase + unc[m * K + min(static_cast<int>(threadIdx.x & 15), nu - 1)] * nov;
  chunk_dots(Vp + md.vbase, nov, nb, w, nu, chunk_begin(nov, ch), chunk_begin(nov, ch + 1),
             part + (static_cast<long>(m) * kXChunks + ch) * kPartStride, L);
}

// ... then the update of chunk c: h = the inner products summed over the
// chunks in order, w_u -= sum_s h[s][u] V_s for the nu <= NR corrections.
template <int NR>
__global__ void __launch_bounds__(256) gs_update_kernel(const MolDesc* __restrict__ mols, int K,
                                                        const double* __restrict__ Vp, double* __restrict__ Wcp,
                                                        const int* __restrict__ S, const int* __restrict__ knew,
                                                        const int* __restrict__ active, const int* __restrict__ coll,
                                                        const int* __restrict__ qcol, const int* __restrict__ unc,
                                                        const double* __restrict__ part) {
  __shared__ double h[kBatchMaxSub][NR];
  const int m = blockIdx.x, ch = blockIdx.y;
  if (!active[m]) return;
  const MolDesc md = mols[m];
  const long nov = md.nov, x0 = chunk_begin(nov, ch), x1 = chunk_begin(nov, ch + 1);
  const int nch = chunks_of(nov);
  if (ch >= nch) return;
  const int nb = coll[m] ? qcol[m] : S[m];
  const int nu = knew[m];
  const double* P = part + static_cast<long>(m) * kXChunks * kPartStride;
  for (int idx = threadIdx.x; idx < kBatchMaxSub * NR; idx += 256) {
    const int sidx = idx / NR, u = idx % NR;
    double d = 0.0;
    if (sidx < nb && u < nu)
      for (int c = 0; c < nch; ++c) d += P[c * kPartStride + sidx * 2 * kBatchMaxRoots + u];
    h[sidx][u] = -d;
  }
  __syncthreads();
  double* w[NR];
#pragma unroll
  for (int u = 0; u < NR; ++u) w[u] = Wcp + md.xbase + unc[m * K + min(u, nu - 1)] * nov;
  for (long x = x0 + threadIdx.x; x < x1; x += 256) {
    double t[NR];
#pragma unroll
    for (int u = 0; u < NR; ++u) t[u] = u < nu ? w[u][x] : 0.0;
    combine_at<NR>(Vp + md.vbase, nov, nb, x, h, t);
#pragma unroll
    for (int u = 0; u < NR; ++u)
      if (u < nu) w[u][x] = t[u];
  }
}

// Orthonormalise the deflated corrections among themselves (modified
// Gram-Schmidt, twice) and append the survivors (norm above 1e-8 of the
// correction's norm before deflation) to the basis.  The pass that takes one
// direction out also forms the inner product with the next (or the norm at the
// end), so each costs one pass and one workgroup sum; a thread always holds the
// same entries, so no barrier orders the passes.
constexpr int kAppendThreads = 512;
__global__ void __launch_bounds__(kAppendThreads) append_kernel(const MolDesc* __restrict__ mols, int K, int Smax,
                                                     double* __restrict__ Vp, double* __restrict__ Wcp, int* S,
                                                     int* knew, int* active, int* coll, const int* __restrict__ qcol,
                                                     const int* __restrict__ unc, int* conv,
                                                     const int* __restrict__ counters,
                                                     const double* __restrict__ n0part) {
  __shared__ double red[2][kAppendThreads / 64];
  const int m = blockIdx.x;
  if (!active[m]) return;
  const MolDesc md = mols[m];
  const long nov = md.nov;
  const int S0 = coll[m] ? qcol[m] : S[m];
  const int nu = knew[m], nch = chunks_of(nov);
  double* V = Vp + md.vbase + static_cast<long>(S0) * nov;
  int acc = 0, turn = 0;
  auto sum = [&](double v) {  // over the workgroup, fixed order; two slots in turn need one barrier a sum
    double* r = red[turn ^= 1];
    v = wave_sum64(v);
    if ((threadIdx.x & 63) == 0) r[threadIdx.x >> 6] = v;
    __syncthreads();
    v = 0.0;
    for (int q = 0; q < kAppendThreads / 64; ++q) v += r[q];
    return v;
  };
  for (int u = 0; u < nu; ++u) {
    if (S0 + acc >= Smax) break;
    double* w = Wcp + md.xbase + unc[m * K + u] * nov;
    double d = 0.0;
    for (long x = threadIdx.x; x < nov; x += kAppendThreads) d += w[x] * (acc > 0 ? V[x] : w[x]);
    d = sum(d);
    for (int i = 0; i < 2 * acc; ++i) {
      const double* a = V + static_cast<long>(i % acc) * nov;
      const double* next = i + 1 < 2 * acc ? V + static_cast<long>((i + 1) % acc) * nov : w;
      double dn = 0.0;
      for (long x = threadIdx.x; x < nov; x += kAppendThreads) {
        const double wx = w[x] - d * a[x];
        w[x] = wx;
        dn += wx * next[x];
      }
      d = sum(dn);
    }
    const double nw = sqrt(d);
    double n02 = 0.0;
    for (int c = 0; c < nch; ++c) n02 += n0part[(static_cast<long>(m) * kXChunks + c) * kBatchMaxRoots + u];
    if (nw > 1e-8 * sqrt(n02) && nw > 1e-14) {
      double* dst = V + static_cast<long>(acc) * nov;
      const double inv = 1.0 / nw;
      for (long x = threadIdx.x; x < nov; x += kAppendThreads) dst[x] = w[x] * inv;
      ++acc;
    }
  }
  __syncthreads();  // S, knew and coll have been read by every wavefront
  if (threadIdx.x == 0) {
    S[m] = S0;
    coll[m] = 0;
    knew[m] = acc;
    if (acc == 0) {  // no new direction: stop this molecule (flagged by a negative iteration)
      active[m] = 0;
      conv[m] = -counters[2];
    }
  }
}

// Amplitudes and properties of every root of every molecule, one workgroup an
// item: X with its largest element (lowest index on ties) positive, Y = 0, the
// transition dipole and the oscillator strength.  Only the same-atom elements
// of the transition density C_o X C_v^T enter the dipole, so T = C_o X is
// formed whole (in the workgroup's slice of scratch, n x v) and its product with
// C_v^T for those alone.  512 molecules, 5 roots: 280 us, where seven launches, two
// copies and a wait for each molecule took 28 ms.
__global__ void __launch_bounds__(kSigThreads) finalize_items_kernel(int nitem, int K, const MolDesc* __restrict__ mols,
                                                             const RootOut* __restrict__ outs,
                                                             const double* __restrict__ Xp,
                                                             const double* __restrict__ omega, double* scratch,
                                                             long scratch_stride) {
  __shared__ double bv[kSigThreads / 64];
  __shared__ long bi[kSigThreads / 64];
  __shared__ double red[3][kSigThreads / 64];
  constexpr int kWaves = kSigThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  double* T = scratch + blockIdx.x * scratch_stride;
  for (int it = blockIdx.x; it < nitem; it += gridDim.x) {
    const int m = it / K, j = it % K;
    const MolDesc md = mols[m];
    const RootOut out = outs[m];
    const long nov = md.nov;
    const int n = md.n, o = md.o, v = md.v;
    const double* x = Xp + md.xbase + j * nov;
    double best = -1.0;
    long at = nov;
    for (long t = tid; t < nov; t += kSigThreads) {
      const double a = fabs(x[t]);
      if (a > best) {  // a strided scan visits indices in increasing order
        best = a;
        at = t;
      }
    }
#pragma unroll
    for (int h = 1; h < 64; h <<= 1) {
      const double a = __shfl_xor(best, h);
      const long ia = __shfl_xor(at, h);
      if (a > best || (a == best && ia < at)) {
        best = a;
        at = ia;
      }
    }
    if (lane == 0) {
      bv[wave] = best;
      bi[wave] = at;
    }
    wg_gemm<double, 2, 1>(n, v, o, md.C64, n, 1, x, v, 1,
                          [&](int i, int c, double t) { T[static_cast<long>(i) * v + c] = t; });
    __syncthreads();
    for (int q = 0; q < kWaves; ++q)
      if (bv[q] > best || (bv[q] == best && bi[q] < at)) {
        best = bv[q];
        at = bi[q];
      }
    const double sign = at < nov && x[at] < 0.0 ? -1.0 : 1.0;
    for (long t = tid; t < nov; t += kSigThreads) {
      out.X[j * nov + t] = sign * x[t];
      out.Y[j * nov + t] = 0.0;
    }
    // one wavefront an atom, lanes over the virtual orbitals
    double s[3] = {0.0, 0.0, 0.0};
    for (int A = wave; A < md.natoms; A += kWaves) {
      const Elem& e = md.elems[md.slot[A]];
      const int a0 = md.ao_off[A], na = e.nao;
      double tr = 0.0, sp[3] = {0.0, 0.0, 0.0};
      for (int c = lane; c < v; c += 64) {
        const double t0 = T[static_cast<long>(a0) * v + c], c0 = md.C64[static_cast<long>(a0) * n + o + c];
        tr += t0 * c0;
        for (int i = 1; i < na; ++i) {
          const double ti = T[static_cast<long>(a0 + i) * v + c], ci = md.C64[static_cast<long>(a0 + i) * n + o + c];
          tr += ti * ci;
          if (na == 4) {
            const double z = t0 * ci + ti * c0;
            sp[0] += i == 1 ? z : 0.0;
            sp[1] += i == 2 ? z : 0.0;
            sp[2] += i == 3 ? z : 0.0;
          }
        }
      }
      tr = wave_sum64(tr);
      for (int c = 0; c < 3; ++c) {
        s[c] += tr * out.xyz[3 * A + c];
        if (na == 4) s[c] += e.D1 * wave_sum64(sp[c]);
      }
    }
    if (lane == 0)
      for (int c = 0; c < 3; ++c) red[c][wave] = s[c];
    __syncthreads();
    if (tid == 0) {
      double m2 = 0.0;
      for (int c = 0; c < 3; ++c) {
        double d = 0.0;
        for (int q = 0; q < kWaves; ++q) d += red[c][q];
        d *= sign * sqrt(2.0);
        out.mu[3 * j + c] = d;
        m2 += d * d;
      }
      const double om = omega[m * K + j];
      out.omega[j] = om;
      out.f[j] = 2.0 / 3.0 * om * m2;
    }
    // bv and red are written again only after the next item's products, T after its own reads ended here
    __syncthreads();
  }
}

int bucket_of(int n) { return n < 32 ? 0 : n < 64 ? 1 : n < 96 ? 2 : n < 128 ? 3 : 4; }

double ms_between(hipEvent_t a, hipEvent_t b) {
  float t = 0.f;
  SEQX_HIP(hipEventElapsedTime(&t, a, b));
  return t;
}

}  // namespace

BatchWork::~BatchWork() {
  if (stream) (void)hipStreamDestroy(stream);
}

BatchResult batched_cis(const std::vector<DeviceMolecule*>& mols, const BatchOptions& opt, BatchWork& w,
                        TileTuning& tune, hipStream_t user_stream) {
  const int nmol = static_cast<int>(mols.size());
  const int K = opt.nroots;
  const bool f32 = opt.precision == kPrecFP32;
  if (opt.precision != kPrecFP32 && opt.precision != kPrecFP64)
    throw Error(kEArg, "batched solve supports FP32 and FP64 products");
  if (K < 1 || K > kBatchMaxRoots) throw Error(kEArg, "batched solve supports 1 to 16 roots");
  int Smax = opt.max_sub > 0 ? opt.max_sub : 8 * K;
  Smax = std::min(std::max(Smax, 3 * K), kBatchMaxSub);
  if (Smax < 3 * K) throw Error(kEArg, "batched solve: subspace cap below 3 * nroots");
  BatchResult res;
  if (!w.stream) SEQX_HIP(hipStreamCreateWithFlags(&w.stream, hipStreamNonBlocking));
  hipStream_t st = w.stream;

  // ---- molecule table, ordering and pools
  std::vector<MolDesc> h(nmol);
  long vtot = 0, xtot = 0, scr = 0;
  int maxnew = 2 * K;
  for (int m = 0; m < nmol; ++m) {
    const DeviceMolecule& d = *mols[m];
    const long nov = static_cast<long>(d.nocc) * d.nvirt;
    if (nov < K) throw Error(kEArg, "nroots exceeds nocc*nvirt of a molecule");
    if (d.np > kBatchMaxNp) throw Error(kEArg, "molecule too large for the batched solver (pair indices > 1536)");
    if (d.C32.n < static_cast<size_t>(d.nao) * d.nao) throw Error(kEState, "FP32 MO coefficients missing");
    MolDesc& md = h[m];
    md.n = d.nao;
    md.o = d.nocc;
    md.v = d.nvirt;
    md.np = d.np;
    md.natoms = d.natoms;
    for (int g = 0; g < 3; ++g) {
      md.npairs[g] = d.npairs[g];
      md.pairs[g] = d.pairs[g].p;
    }
    md.variant = 2;
    md.pad_ = 0;
    md.nov = nov;
    md.vbase = vtot;
    md.xbase = xtot;
    vtot += static_cast<long>(Smax) * nov;
    xtot += static_cast<long>(K) * nov;
    md.C32 = d.C32.p;
    md.C64 = d.C.p;
    md.eps = d.eps.p;
    md.W = d.W.p;
    md.slot = d.slot.p;
    md.ao_off = d.ao_off.p;
    md.pi_off = d.pi_off.p;
    md.pi_mu = d.pi_mu.p;
    md.pi_nu = d.pi_nu.p;
    md.elems = d.elems;
    scr = std::max(scr, 2L * d.nao * d.nao + static_cast<long>(d.nao) * d.nvirt);
  }
  std::vector<int> order(nmol);
  for (int m = 0; m < nmol; ++m) order[m] = m;
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return h[a].n > h[b].n; });

  // persistent grid: as many workgroups as fit on the device at once
  int dev = 0, ncu = 0, occ = 0;
  SEQX_HIP(hipGetDevice(&dev));
  SEQX_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
  if (f32)
    SEQX_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, sigma_items_kernel<float>, kSigThreads, 0));
  else
    SEQX_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, sigma_items_kernel<double>, kSigThreads, 0));
  const int G = std::max(1, ncu * std::max(1, occ));
  const long scr_stride = (scr + 63) / 64 * 64;

  w.mols.ensure(nmol);
  w.order.ensure(nmol);
  w.outs.ensure(nmol);
  for (DBuf<int>* b : {&w.S, &w.knew, &w.active, &w.coll, &w.qcol, &w.conv}) b->ensure(nmol);
  w.unc.ensure(static_cast<size_t>(nmol) * K);
  w.counters.ensure(4);
  w.nsig.ensure(3);
  w.stamps.ensure(2 * static_cast<size_t>(G));
  w.items.ensure(static_cast<size_t>(nmol) * std::max(maxnew, K));
  w.V.ensure(vtot);
  w.AV.ensure(vtot);
  w.X.ensure(xtot);
  w.Wc.ensure(xtot);
  w.Mp.ensure(static_cast<size_t>(nmol) * Smax * Smax);
  w.evec.ensure(static_cast<size_t>(nmol) * Smax * Smax);
  w.eval.ensure(static_cast<size_t>(nmol) * Smax);
  w.omega.ensure(static_cast<size_t>(nmol) * K);
  w.rnorm.ensure(static_cast<size_t>(nmol) * K);
  w.rpart.ensure(static_cast<size_t>(nmol) * kXChunks * kBatchMaxRoots);
  w.part.ensure(static_cast<size_t>(nmol) * kXChunks * kPartStride);
  w.n0.ensure(static_cast<size_t>(nmol) * kXChunks * kBatchMaxRoots);
  if (f32) w.scratch32.ensure(static_cast<size_t>(G) * scr_stride);
  else w.scratch64.ensure(static_cast<size_t>(G) * scr_stride);

  // order against the caller's stream
  hipEvent_t ev_in, ev_a, ev_b;
  SEQX_HIP(hipEventCreate(&ev_in));
  SEQX_HIP(hipEventCreate(&ev_a));
  SEQX_HIP(hipEventCreate(&ev_b));
  auto destroy_events = [&] {
    for (hipEvent_t e : {ev_in, ev_a, ev_b}) (void)hipEventDestroy(e);
  };
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  try {
    SEQX_HIP(hipEventRecord(ev_in, user_stream));
    SEQX_HIP(hipStreamWaitEvent(st, ev_in, 0));
    SEQX_HIP(hipMemcpyAsync(w.order.p, order.data(), nmol * sizeof(int), hipMemcpyHostToDevice, st));
    std::vector<int> zero4(4, 0);
    SEQX_HIP(hipMemcpyAsync(w.counters.p, zero4.data(), 4 * sizeof(int), hipMemcpyHostToDevice, st));
    const long long z3[3] = {0, 0, 0};
    SEQX_HIP(hipMemcpyAsync(w.nsig.p, z3, 3 * sizeof(long long), hipMemcpyHostToDevice, st));

    auto upload_desc = [&] {
      SEQX_HIP(hipMemcpyAsync(w.mols.p, h.data(), nmol * sizeof(MolDesc), hipMemcpyHostToDevice, st));
    };
    auto launch_sigma = [&] {
      if (f32)
        hipLaunchKernelGGL(sigma_items_kernel<float>, dim3(G), dim3(kSigThreads), 0, st, w.mols.p, w.items.p, w.counters.p,
                           w.V.p, w.AV.p, w.scratch32.p, scr_stride, w.stamps.p);
      else
        hipLaunchKernelGGL(sigma_items_kernel<double>, dim3(G), dim3(kSigThreads), 0, st, w.mols.p, w.items.p, w.counters.p,
                           w.V.p, w.AV.p, w.scratch64.p, scr_stride, w.stamps.p);
      SEQX_LAUNCH_CHECK();
    };

    // ---- autotuner: per size bucket, time each tile variant on the bucket's molecules
    const int pk = f32 ? 0 : 1;
    std::vector<int> bucket(nmol);
    for (int m = 0; m < nmol; ++m) bucket[m] = bucket_of(h[m].n);
    upload_desc();
    hipLaunchKernelGGL(guess_kernel, dim3(nmol), dim3(256), 0, st, nmol, w.mols.p, K, w.V.p, w.S.p, w.knew.p,
                       w.active.p, w.conv.p, w.coll.p, w.qcol.p);
    SEQX_LAUNCH_CHECK();
    const auto ta0 = std::chrono::steady_clock::now();
    for (int b = 0; b < kNumSizeBuckets; ++b) {
      std::vector<int> mb;
      for (int m = 0; m < nmol; ++m)
        if (bucket[m] == b) mb.push_back(m);
      if (mb.empty()) continue;
      if (!opt.autotune) {
        tune.best[pk][b] = 2;
        continue;
      }
      if (tune.tuned[pk][b]) continue;
      // sample: up to 2 G items of this bucket (the first one or two guess vectors)
      std::vector<int2> it;
      for (int m : mb)
        for (int j = 0; j < std::min<long>(2, h[m].nov) && static_cast<int>(it.size()) < 2 * G; ++j)
          it.push_back(make_int2(m, j));
      const int ni = static_cast<int>(it.size());
      SEQX_HIP(hipMemcpyAsync(w.items.p, it.data(), ni * sizeof(int2), hipMemcpyHostToDevice, st));
      SEQX_HIP(hipMemcpyAsync(w.counters.p, &ni, sizeof(int), hipMemcpyHostToDevice, st));
      double best = 1e300;
      for (int var = 0; var < kNumTileVariants; ++var) {
        for (int m : mb) h[m].variant = var;
        upload_desc();
        launch_sigma();  // warm-up
        SEQX_HIP(hipEventRecord(ev_a, st));
        for (int rep = 0; rep < 3; ++rep) launch_sigma();
        SEQX_HIP(hipEventRecord(ev_b, st));
        SEQX_HIP(hipEventSynchronize(ev_b));
        const double t = ms_between(ev_a, ev_b) / 3.0;
        tune.ms[pk][b][var] = t;
        if (t < best) {
          best = t;
          tune.best[pk][b] = var;
        }
      }
      tune.tuned[pk][b] = true;
    }
    res.t_autotune_ms = 1e3 * std::chrono::duration<double>(std::chrono::steady_clock::now() - ta0).count();
    for (int m = 0; m < nmol; ++m) h[m].variant = tune.best[pk][bucket[m]];
    for (int b = 0; b < kNumSizeBuckets; ++b) res.variant_of_bucket[b] = tune.best[pk][b];
    upload_desc();
    SEQX_HIP(hipMemcpyAsync(w.counters.p, zero4.data(), 4 * sizeof(int), hipMemcpyHostToDevice, st));

    // ---- one iteration as a fixed launch sequence
    const int Q = 2 * K;
    // The projected eigenproblems: K pairs, and the 2K of a collapse where the
    // new directions may not fit.  One Jacobi solve of all pairs in LDS, started
    // from the previous vectors, took 430 us an iteration however few molecules
    // were left; the lowest pairs by reduction and inverse iteration take 205 (65
    // + 100 + 40) with all 512 molecules or few.  Their
    // scratch is the partial inner products' (free between project and gs_dots).
    const EigBatch eig{Smax, K, Q, static_cast<long>(kXChunks) * kPartStride, w.S.p, w.active.p,
                       w.Mp.p, w.evec.p, w.eval.p, w.part.p};
    auto iteration = [&](bool timed) {
      hipLaunchKernelGGL(items_kernel, dim3(1), dim3(256), 0, st, nmol, w.mols.p, w.order.p, w.S.p, w.knew.p,
                         w.active.p, w.items.p, w.counters.p, w.nsig.p);
      launch_sigma();
      if (timed) hipLaunchKernelGGL(stamp_span_kernel, dim3(1), dim3(256), 0, st, G, w.stamps.p, w.nsig.p + 1);
      hipLaunchKernelGGL(project_part_kernel, dim3(nmol, kXChunks), dim3(256), 0, st, w.mols.p, w.V.p, w.AV.p,
                         w.S.p, w.knew.p, w.active.p, w.part.p);
      hipLaunchKernelGGL(project_kernel, dim3(nmol), dim3(256), 0, st, w.mols.p, Smax, w.part.p, w.Mp.p, w.S.p, w.knew.p,
                         w.active.p);
      hipLaunchKernelGGL(advance_kernel, dim3(ceil_div(nmol, 256)), dim3(256), 0, st, nmol, w.S.p, w.knew.p,
                         w.active.p);
      launch_eig_batch(st, nmol, eig);
      // kernels for at least the K roots wanted (registers for each of them)
      const auto rest = [&](auto nr) {
        constexpr int NR = decltype(nr)::value;
        const dim3 chunks(nmol, kXChunks);
        hipLaunchKernelGGL(ritz_kernel<NR>, chunks, dim3(256), 0, st, w.mols.p, K, Smax, w.V.p, w.AV.p, w.evec.p,
                           w.eval.p, w.S.p, w.active.p, w.X.p, w.Wc.p, w.omega.p, w.rpart.p);
        hipLaunchKernelGGL(select_kernel, dim3(1), dim3(256), 0, st, nmol, w.mols.p, K, Smax, opt.tol, w.rpart.p,
                           w.rnorm.p, w.S.p, w.knew.p, w.active.p, w.coll.p, w.qcol.p, w.unc.p, w.conv.p,
                           w.counters.p);
        hipLaunchKernelGGL(collapse_kernel<2 * NR>, chunks, dim3(256), 0, st, w.mols.p, Smax, w.V.p, w.AV.p, w.evec.p,
                           w.eval.p, w.S.p, w.coll.p, w.qcol.p, w.Mp.p);
        hipLaunchKernelGGL(precond_kernel, chunks, dim3(256), 0, st, w.mols.p, K, w.Wc.p, w.knew.p, w.active.p,
                           w.unc.p, w.omega.p, w.n0.p);
        for (int pass = 0; pass < 2; ++pass) {
          hipLaunchKernelGGL(gs_dots_kernel, chunks, dim3(256), 0, st, w.mols.p, K, w.V.p, w.Wc.p, w.S.p, w.knew.p,
                             w.active.p, w.coll.p, w.qcol.p, w.unc.p, w.part.p);
          hipLaunchKernelGGL(gs_update_kernel<NR>, chunks, dim3(256), 0, st, w.mols.p, K, w.V.p, w.Wc.p, w.S.p,
                             w.knew.p, w.active.p, w.coll.p, w.qcol.p, w.unc.p, w.part.p);
        }
      };
      if (K <= 3) rest(std::integral_constant<int, 3>{});
      else if (K <= 5) rest(std::integral_constant<int, 5>{});
      else if (K <= 8) rest(std::integral_constant<int, 8>{});
      else if (K <= 12) rest(std::integral_constant<int, 12>{});
      else rest(std::integral_constant<int, 16>{});
      hipLaunchKernelGGL(append_kernel, dim3(nmol), dim3(kAppendThreads), 0, st, w.mols.p, K, Smax, w.V.p, w.Wc.p,
                         w.S.p, w.knew.p, w.active.p, w.coll.p, w.qcol.p, w.unc.p, w.conv.p, w.counters.p, w.n0.p);
      SEQX_LAUNCH_CHECK();
    };
    if (opt.graph) {
      // capture one iteration; if the runtime refuses any step, run eagerly instead
      bool ok = hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal) == hipSuccess;
      if (ok) {
        try {
          iteration(true);
        } catch (const Error&) {
          ok = false;
        }
        hipGraph_t g = nullptr;
        const hipError_t e = hipStreamEndCapture(st, &g);
        graph = g;
        ok = ok && e == hipSuccess && graph != nullptr;
        ok = ok && hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) == hipSuccess;
        (void)hipGetLastError();
      }
      if (!ok) {
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
        exec = nullptr;
        graph = nullptr;
      }
      res.used_graph = ok;
    }
    SEQX_HIP(hipEventRecord(ev_a, st));
    int it = 0, counters[4] = {0, 0, 0, 0};
    for (it = 1; it <= opt.max_iter; ++it) {
      if (exec) SEQX_HIP(hipGraphLaunch(exec, st));
      else iteration(true);
      SEQX_HIP(hipMemcpyAsync(counters, w.counters.p, 4 * sizeof(int), hipMemcpyDeviceToHost, st));
      SEQX_HIP(hipStreamSynchronize(st));
      if (counters[1] == 0) break;
    }
    SEQX_HIP(hipEventRecord(ev_b, st));
    SEQX_HIP(hipEventSynchronize(ev_b));
    res.t_solve_ms = ms_between(ev_a, ev_b);
    res.iterations = std::min(it, opt.max_iter);
    long long ns[3] = {0, 0, 0};
    res.conv_iter.resize(nmol);
    SEQX_HIP(hipMemcpyAsync(ns, w.nsig.p, 3 * sizeof(long long), hipMemcpyDeviceToHost, st));
    SEQX_HIP(hipMemcpyAsync(res.conv_iter.data(), w.conv.p, nmol * sizeof(int), hipMemcpyDeviceToHost, st));
    SEQX_HIP(hipStreamSynchronize(st));
    res.n_sigma = ns[0];
    res.sigma_flops = static_cast<double>(ns[2]);
    int rate_khz = 0;  // device wall clock (the stamps of the sigma launches)
    if (hipDeviceGetAttribute(&rate_khz, hipDeviceAttributeWallClockRate, dev) == hipSuccess && rate_khz > 0)
      res.t_sigma_ms = static_cast<double>(ns[1]) / rate_khz;
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    exec = nullptr;
    graph = nullptr;
    for (int m = 0; m < nmol; ++m)
      if (res.conv_iter[m] <= 0)
        throw Error(kEDavNoConv, res.conv_iter[m] < 0 ? "batched Davidson: no new direction for a molecule"
                                                      : "batched Davidson did not converge in " +
                                                            std::to_string(opt.max_iter) + " iterations");
    // ---- amplitudes and properties of all molecules, on the caller's stream
    SEQX_HIP(hipEventRecord(ev_b, st));
    SEQX_HIP(hipStreamWaitEvent(user_stream, ev_b, 0));
    std::vector<RootOut> outs(nmol);
    for (int m = 0; m < nmol; ++m) {
      DeviceMolecule& d = *mols[m];
      d.omega.ensure(K);
      d.X.ensure(static_cast<size_t>(K) * h[m].nov);
      d.Y.ensure(static_cast<size_t>(K) * h[m].nov);
      d.f.ensure(K);
      d.mu.ensure(3 * K);
      outs[m] = RootOut{d.X.p, d.Y.p, d.omega.p, d.f.p, d.mu.p, d.xyz.p};
    }
    SEQX_HIP(hipMemcpyAsync(w.outs.p, outs.data(), nmol * sizeof(RootOut), hipMemcpyHostToDevice, user_stream));
    // a slice holds 2 n^2 + n v elements of the products' type, at least n v doubles
    double* slices = f32 ? reinterpret_cast<double*>(w.scratch32.p) : w.scratch64.p;
    hipLaunchKernelGGL(finalize_items_kernel, dim3(std::min(G, nmol * K)), dim3(kSigThreads), 0, user_stream, nmol * K,
                       K, w.mols.p, w.outs.p, w.X.p, w.omega.p, slices, f32 ? scr_stride / 2 : scr_stride);
    SEQX_LAUNCH_CHECK();
    SEQX_HIP(hipStreamSynchronize(user_stream));
    for (int m = 0; m < nmol; ++m) {
      mols[m]->nroots = K;
      mols[m]->theory = 0;
      mols[m]->dav_iterations = res.conv_iter[m];
    }
  } catch (...) {
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    (void)hipStreamSynchronize(st);
    destroy_events();
    throw;
  }
  destroy_events();
  return res;
}

}  // namespace seqx
