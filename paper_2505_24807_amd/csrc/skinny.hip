// Tall-skinny FP64 products of the Davidson iteration on the CDNA4 matrix
// cores: inner products of a few vectors with a long basis (split over chunks
// of the vector length, partial sums reduced in a fixed order) and
// combinations of a basis into a few vectors.
#include <algorithm>
#include <type_traits>

#include "gemm.hpp"

namespace seqx {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

bool aligned_to(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// Tall-skinny combinations on the FP64 matrix cores: C[m][x] = alpha sum_s
// A[m][s] B[s][x] + beta C[m][x] for M <= 48 rows and long rows x (new
// Davidson vectors as combinations of the basis).  A wavefront owns every row
// and 64 columns (four 16-column tiles); B is read once, in 128-byte row
// segments per tile; the operands of the next k-step are loaded before the
// MFMAs of the current one.
template <int NX, class TB, class TC>
__global__ void __launch_bounds__(256) skinny_combine_kernel(int M, long N, int K, double alpha,
                                                             const double* __restrict__ A, long lda,
                                                             const TB* __restrict__ B, long ldb, double beta,
                                                             TC* __restrict__ C, long ldc) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = lane & 15, g = lane >> 4;
  const long x0 = (static_cast<long>(blockIdx.x) * 4 + wave) * 64;
  if (x0 >= N) return;
  long xc[4];  // this lane's column in each tile (clamped; columns past N are not stored)
#pragma unroll
  for (int b = 0; b < 4; ++b) xc[b] = min(x0 + 16 * b + i, N - 1);
  const double* ar[NX];
#pragma unroll
  for (int a = 0; a < NX; ++a) ar[a] = A + static_cast<long>(min(16 * a + i, M - 1)) * lda;
  d4 acc[NX][4];
#pragma unroll
  for (int a = 0; a < NX; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = d4{0, 0, 0, 0};
  const int nfull = K / 4;
  auto load = [&](int step, double* av, double* bv) {
    const int sk = 4 * step + g;
#pragma unroll
    for (int a = 0; a < NX; ++a) av[a] = ar[a][sk];
    const TB* brow = B + static_cast<long>(sk) * ldb;
#pragma unroll
    for (int b = 0; b < 4; ++b) bv[b] = static_cast<double>(brow[xc[b]]);
  };
  auto mma = [&](const double* av, const double* bv) {
#pragma unroll
    for (int a = 0; a < NX; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
  };
  if (nfull > 0) {
    double a0[NX], b0[4], a1[NX], b1[4];
    load(0, a0, b0);
    int st = 0;
    for (; st + 1 < nfull; st += 2) {
      load(st + 1, a1, b1);
      mma(a0, b0);
      load(min(st + 2, nfull - 1), a0, b0);
      mma(a1, b1);
    }
    if (st < nfull) mma(a0, b0);
  }
  if (4 * nfull < K) {  // k tail: slots past K are zero
    const int sk = 4 * nfull + g;
    const bool in = sk < K;
    double av[NX], bv[4];
#pragma unroll
    for (int a = 0; a < NX; ++a) av[a] = in ? ar[a][sk] : 0.0;
    const TB* brow = B + static_cast<long>(in ? sk : 0) * ldb;
#pragma unroll
    for (int b = 0; b < 4; ++b) bv[b] = in ? static_cast<double>(brow[xc[b]]) : 0.0;
    mma(av, bv);
  }
#pragma unroll
  for (int a = 0; a < NX; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = 16 * a + g + 4 * r;
        const long x = x0 + 16 * b + i;
        if (m < M && x < N) {
          TC* cp = C + static_cast<long>(m) * ldc + x;
          const double v = alpha * acc[a][b][r];
          *cp = static_cast<TC>(beta == 0.0 ? v : v + beta * static_cast<double>(*cp));
        }
      }
}

// sum over the chunks of the partial sums: a workgroup takes 64 outputs (one
// per lane, coalesced) and splits the chunks over its 16 wavefronts (wavefront
// w: chunks w, w + 16, ..., four independent running sums), then adds the 16
// wavefront sums in order, so the result does not depend on timing
constexpr int kRedWaves = 16;
__global__ void __launch_bounds__(64 * kRedWaves) reduce_partials_kernel(int nchunks, int ns, int nt,
                                                                          const double* __restrict__ part, double* out,
                                                                          long ldo) {
  __shared__ double red[kRedWaves][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int idx = blockIdx.x * 64 + lane;
  const long stride = static_cast<long>(ns) * nt;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  if (idx < ns * nt) {
    const double* p = part + idx;
    int c = wave;
    for (; c + 3 * kRedWaves < nchunks; c += 4 * kRedWaves) {
      a0 += p[c * stride];
      a1 += p[(c + kRedWaves) * stride];
      a2 += p[(c + 2 * kRedWaves) * stride];
      a3 += p[(c + 3 * kRedWaves) * stride];
    }
    for (; c < nchunks; c += kRedWaves) a0 += p[c * stride];
  }
  red[wave][lane] = (a0 + a1) + (a2 + a3);
  __syncthreads();
  if (wave == 0 && idx < ns * nt) {
    double acc = 0.0;
#pragma unroll
    for (int w = 0; w < kRedWaves; ++w) acc += red[w][lane];
    out[static_cast<long>(idx / nt) * ldo + idx % nt] = acc;
  }
}

// few outputs, many chunks: one workgroup per output, fixed-order tree
__global__ void __launch_bounds__(256) reduce_partials_wide_kernel(int nchunks, int ns, int nt,
                                                                   const double* __restrict__ part, double* out,
                                                                   long ldo) {
  __shared__ double red[256];
  const int idx = blockIdx.x;
  const long stride = static_cast<long>(ns) * nt;
  double acc = 0.0;
  for (int c = threadIdx.x; c < nchunks; c += 256) acc += part[c * stride + idx];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[static_cast<long>(idx / nt) * ldo + idx % nt] = red[0];
}

}  // namespace

template <class TB, class TC>
void combine_pass(hipStream_t st, int M, long N, int K, double alpha, const double* A, long lda, const TB* B,
                  long ldb, double beta, TC* C, long ldc) {
  const dim3 grid(static_cast<unsigned>((N + 255) / 256));
  if (M <= 16)
    hipLaunchKernelGGL((skinny_combine_kernel<1, TB, TC>), grid, dim3(256), 0, st, M, N, K, alpha, A, lda, B, ldb,
                       beta, C, ldc);
  else if (M <= 32)
    hipLaunchKernelGGL((skinny_combine_kernel<2, TB, TC>), grid, dim3(256), 0, st, M, N, K, alpha, A, lda, B, ldb,
                       beta, C, ldc);
  else
    hipLaunchKernelGGL((skinny_combine_kernel<3, TB, TC>), grid, dim3(256), 0, st, M, N, K, alpha, A, lda, B, ldb,
                       beta, C, ldc);
  SEQX_LAUNCH_CHECK();
}

void skinny_combine(hipStream_t st, int M, long N, int K, double alpha, const double* A, long lda, const double* B,
                    long ldb, double beta, double* C, long ldc) {
  combine_pass<double, double>(st, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc);
}

template <class TB, class TC>
void combine_rows(hipStream_t st, int M, long N, int K, double alpha, const double* A, long lda, const TB* B, long ldb,
                  double beta, TC* C, long ldc) {
  if (M <= 0 || N <= 0) return;
  for (int r0 = 0; r0 < M; r0 += 48)
    combine_pass<TB, TC>(st, std::min(48, M - r0), N, K, alpha, A + static_cast<long>(r0) * lda, lda, B, ldb, beta,
                         C + static_cast<long>(r0) * ldc, ldc);
}
template void combine_rows<double, double>(hipStream_t, int, long, int, double, const double*, long, const double*,
                                           long, double, double*, long);
template void combine_rows<float, double>(hipStream_t, int, long, int, double, const double*, long, const float*, long,
                                          double, double*, long);
template void combine_rows<double, float>(hipStream_t, int, long, int, double, const double*, long, const double*, long,
                                          double, float*, long);
template void combine_rows<float, float>(hipStream_t, int, long, int, double, const double*, long, const float*, long,
                                         double, float*, long);

// Tall-skinny inner products on the FP64 matrix cores: partial[c][s][t] =
// sum over k in chunk c of X[s][k] Y[t][k], for ns <= 48 rows of X and any
// number of rows of Y (the Davidson basis).  A workgroup takes every row of X
// and 128 rows of Y (32 per wavefront) over one chunk of k (a multiple of 16,
// chosen so that the grid holds about a thousand workgroups), so Y is read
// once.  Within each block of 16 k-values lane l loads the 4
// contiguous values 4 (l / 16) .. +3 of its rows (row l % 16 of each 16-row
// tile) as two 16-byte loads; MFMA step q then takes value q, i.e. k-slot
// l / 16 of step q is k = 4 (l / 16) + q.  The sum over k is the same whatever
// slot holds which k, so no operand has to be rearranged through LDS.
namespace {


// 4 contiguous values (16-byte aligned) as doubles
__device__ __forceinline__ void load4(const double* p, double* o) {
  const d2 a = *reinterpret_cast<const d2*>(p), b = *reinterpret_cast<const d2*>(p + 2);
  o[0] = a[0];
  o[1] = a[1];
  o[2] = b[0];
  o[3] = b[1];
}
__device__ __forceinline__ void load4(const float* p, double* o) {
  typedef float f4v __attribute__((ext_vector_type(4)));
  const f4v a = *reinterpret_cast<const f4v*>(p);
  o[0] = a[0];
  o[1] = a[1];
  o[2] = a[2];
  o[3] = a[3];
}

// 4 contiguous values whose address is only a multiple of the element size
template <class T>
__device__ __forceinline__ void load4_any(const T* p, double* o) {
#pragma unroll
  for (int q = 0; q < 4; ++q) o[q] = static_cast<double>(p[q]);
}

// X and Y rows of FP64 or FP32 elements (FP32 ones widened on load); FP64
// products.
//   kRowsAligned: row starts are 16-byte aligned.
//   kRowsAny: they are not (an odd row length, as in C40H42 with nov = 101 *
//     101); the same four values per lane come as four element loads, which hit
//     the same cache lines.
//   kRowsOne: a single short row of X, one chunk over all of it with k in
//     ascending order (MFMA step q of a block takes k = 4 q + l / 16) and one
//     16-row tile of Y per wavefront.  The Coulomb part of every SCF below 1024
//     same-atom pairs comes from here: the order of its sums is part of the
//     reproducible orbitals.
enum DotRows { kRowsAligned, kRowsAny, kRowsOne };

template <int NX, class TX, class TY, int ROWS>
__global__ void __launch_bounds__(256) skinny_dots_kernel(int ns, int nt, const TX* __restrict__ X, long ldx,
                                                          const TY* __restrict__ Y, long ldy, long len,
                                                          long chunk, double* __restrict__ part) {
  constexpr int NB = ROWS == kRowsOne ? 1 : 2;  // 16-row tiles of Y per wavefront
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = lane & 15, g = lane >> 4;
  const int t0 = (blockIdx.x * 4 + wave) * (16 * NB);
  const long k0 = static_cast<long>(blockIdx.y) * chunk;
  const long k1 = k0 + chunk < len ? k0 + chunk : len;
  if (t0 >= nt) return;
  // rows of this lane (clamped: rows past ns / nt feed outputs that are not stored)
  const TX* xr[NX];
#pragma unroll
  for (int a = 0; a < NX; ++a) xr[a] = X + static_cast<long>(min(16 * a + i, ns - 1)) * ldx;
  const TY* yr[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) yr[b] = Y + static_cast<long>(min(t0 + 16 * b + i, nt - 1)) * ldy;
  d4 acc[NX][NB];
#pragma unroll
  for (int a = 0; a < NX; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = d4{0, 0, 0, 0};
  // blocks of 16 k-values; the loads of block + 1 are issued before the MFMAs
  // of the current block (past the last full block they repeat it)
  const long nfull = (k1 - k0) / 16;
  auto load = [&](long blk, double (*xv)[4], double (*yv)[4]) {
    const long kk = k0 + 16 * blk + (ROWS == kRowsOne ? g : 4 * g);
#pragma unroll
    for (int a = 0; a < NX; ++a) {
      if constexpr (ROWS == kRowsAligned) load4(xr[a] + kk, xv[a]);
      else if constexpr (ROWS == kRowsAny) load4_any(xr[a] + kk, xv[a]);
      else
#pragma unroll
        for (int q = 0; q < 4; ++q) xv[a][q] = static_cast<double>(xr[a][kk + 4 * q]);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if constexpr (ROWS == kRowsAligned) load4(yr[b] + kk, yv[b]);
      else if constexpr (ROWS == kRowsAny) load4_any(yr[b] + kk, yv[b]);
      else
#pragma unroll
        for (int q = 0; q < 4; ++q) yv[b][q] = static_cast<double>(yr[b][kk + 4 * q]);
    }
  };
  auto mma = [&](double (*xv)[4], double (*yv)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int a = 0; a < NX; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(xv[a][q], yv[b][q], acc[a][b], 0, 0, 0);
  };
  if (nfull > 0) {
    double xa0[NX][4], ya0[NB][4], xa1[NX][4], ya1[NB][4];
    load(0, xa0, ya0);
    long blk = 0;
    for (; blk + 1 < nfull; blk += 2) {
      load(blk + 1, xa1, ya1);
      mma(xa0, ya0);
      load(min(blk + 2, nfull - 1), xa0, ya0);
      mma(xa1, ya1);
    }
    if (blk < nfull) mma(xa0, ya0);
  }
  long k = k0 + 16 * nfull;
  if (k < k1) {  // ragged end of the last chunk: element loads, zero past len
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const long kk = ROWS == kRowsOne ? k + 4 * q + g : k + 4 * g + q;
      const bool in = kk < k1;
#pragma unroll
      for (int a = 0; a < NX; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? static_cast<double>(xr[a][kk]) : 0.0,
                                                           in ? static_cast<double>(yr[b][kk]) : 0.0, acc[a][b], 0,
                                                           0, 0);
    }
  }
  double* out = part + static_cast<long>(blockIdx.y) * ns * nt;
#pragma unroll
  for (int a = 0; a < NX; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int s = 16 * a + (lane >> 4) + 4 * r, t = t0 + 16 * b + (lane & 15);
        if (s < ns && t < nt) out[static_cast<long>(s) * nt + t] = acc[a][b][r];
      }
}

}  // namespace

// Chunk length: about 1024 workgroups, at least 256 values.  Rows below 1024
// values take chunks of 64 (4 MFMA blocks a wavefront): one molecule of 30-90
// AOs gives only a handful of 128-row groups, and the short chunks keep the
// serial part near a microsecond.
constexpr long kShortDot = 1024;
long skinny_chunk(int nt, long len) {
  const long groups = (nt + 127) / 128;
  const long want = std::max<long>(1, 1024 / groups);
  long chunk = (len + want - 1) / want;
  chunk = (chunk + 15) / 16 * 16;
  return std::max<long>(chunk, len < kShortDot ? 64 : 256);
}

// Rows of X per pass of the inner products: the tall-skinny kernels hold at
// most 48 rows; more rows take several passes, each reading Y once.
constexpr int kDotRows = 48;

// Partial sums of one pass of at most kDotRows rows: whatever nt is, at most 16
// chunks of a vector below kShortDot and min(1024, len / 256) above.  The bound
// is monotone in ns, nt and len: a workspace sized for the largest shape serves
// every smaller one.
size_t dots_workspace(int ns, int nt, long len) {
  const long nchunks = std::max(std::min<long>(16, (len + 63) / 64), std::min<long>(1024, (len + 255) / 256));
  return static_cast<size_t>(nchunks) * std::min(ns, kDotRows) * nt;
}

namespace {

// rows whose starts are 16-byte aligned (the loads then take 4 contiguous values)
template <class TX, class TY>
bool rows_aligned(const TX* X, long ldx, const TY* Y, long ldy) {
  const long ax = 16 / sizeof(TX), ay = 16 / sizeof(TY);
  return ldx % ax == 0 && ldy % ay == 0 && aligned_to(X, 16) && aligned_to(Y, 16);
}

template <class TX, class TY, int ROWS>
void dots_pass(hipStream_t st, int ns, const TX* X, long ldx, int nt, const TY* Y, long ldy, long len, double* out,
               long ldo, double* ws) {
  const long chunk = ROWS == kRowsOne ? len : skinny_chunk(nt, len);
  const int nchunks = static_cast<int>((len + chunk - 1) / chunk);
  const dim3 grid(ceil_div(nt, ROWS == kRowsOne ? 64 : 128), nchunks);
  const auto launch = [&](auto nx) {
    hipLaunchKernelGGL((skinny_dots_kernel<decltype(nx)::value, TX, TY, ROWS>), grid, dim3(256), 0, st, ns, nt, X, ldx,
                       Y, ldy, len, chunk, ws);
  };
  if constexpr (ROWS == kRowsOne) launch(std::integral_constant<int, 1>{});
  else if (ns <= 16) launch(std::integral_constant<int, 1>{});
  else if (ns <= 32) launch(std::integral_constant<int, 2>{});
  else launch(std::integral_constant<int, 3>{});
  if (ns * nt < 1024 && nchunks >= 64)
    hipLaunchKernelGGL(reduce_partials_wide_kernel, dim3(ns * nt), dim3(256), 0, st, nchunks, ns, nt, ws, out, ldo);
  else
    hipLaunchKernelGGL(reduce_partials_kernel, dim3(ceil_div(ns * nt, 64)), dim3(64 * kRedWaves), 0, st, nchunks, ns,
                       nt, ws, out, ldo);
  SEQX_LAUNCH_CHECK();
}

}  // namespace

// Any length and alignment.  Products over 804 same-atom pairs ((H2O)67, 7
// vectors) took 110 us as a general GEMM of 7 x 804 outputs; with the short
// and odd rows on these kernels the pass of seven (A+B)V, (A-B)V products
// there went 362 -> 256 us, 20 CIS roots of C40H42 (nov odd) 159 -> 129 ms and
// the parameter derivatives of C20H22 21.8 -> 16.5 ms.
void dots(hipStream_t st, int ns, const double* X, long ldx, int nt, const double* Y, long ldy, long len, double* out,
          long ldo, double* ws) {
  if (ns <= 0 || nt <= 0) return;
  const bool al = rows_aligned(X, ldx, Y, ldy);
  // passes of at most kDotRows rows share the workspace (ordered on st)
  for (int r0 = 0; r0 < ns; r0 += kDotRows) {
    const int nr = std::min(kDotRows, ns - r0);
    const double* Xr = X + static_cast<long>(r0) * ldx;
    double* outr = out + static_cast<long>(r0) * ldo;
    if (ns == 1 && len < kShortDot) dots_pass<double, double, kRowsOne>(st, nr, Xr, ldx, nt, Y, ldy, len, outr, ldo, ws);
    else if (al) dots_pass<double, double, kRowsAligned>(st, nr, Xr, ldx, nt, Y, ldy, len, outr, ldo, ws);
    else dots_pass<double, double, kRowsAny>(st, nr, Xr, ldx, nt, Y, ldy, len, outr, ldo, ws);
  }
}

// Inner products with FP32 rows on either side (widened to FP64 on load, FP64
// products and sums): rows must be long and their starts 16-byte aligned.
template <class TX, class TY>
void dots_mixed(hipStream_t st, int ns, const TX* X, long ldx, int nt, const TY* Y, long ldy, long len, double* out,
                long ldo, double* ws) {
  if (ns <= 0 || nt <= 0) return;
  if (len < 1024 || !rows_aligned(X, ldx, Y, ldy)) throw Error(kEArg, "FP32 inner products need long, 16-byte aligned rows");
  for (int r0 = 0; r0 < ns; r0 += kDotRows)
    dots_pass<TX, TY, kRowsAligned>(st, std::min(kDotRows, ns - r0), X + static_cast<long>(r0) * ldx, ldx, nt, Y, ldy, len,
              out + static_cast<long>(r0) * ldo, ldo, ws);
}
template void dots_mixed<float, float>(hipStream_t, int, const float*, long, int, const float*, long, long, double*,
                                       long, double*);
template void dots_mixed<double, float>(hipStream_t, int, const double*, long, int, const float*, long, long, double*,
                                        long, double*);
template void dots_mixed<float, double>(hipStream_t, int, const float*, long, int, const double*, long, long, double*,
                                        long, double*);

}  // namespace seqx
