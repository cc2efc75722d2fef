// Dense GEMMs on the matrix cores of gfx950, FP64 (v_mfma_f64_16x16x4f64) and
// FP32 (v_mfma_f32_16x16x4f32) inputs.
//
// Each 256-thread block (4 wavefronts of 64) owns a tile of C and walks K in
// steps of 16: the A and B panels are staged through LDS in k-major order so
// that every lane fetches its MFMA operand with one conflict-free read, and
// each wavefront accumulates 16x16 tiles.  Operands: lane l holds A[l%16][l/16]
// and B[l/16][l%16].  Accumulator register r of lane l holds column l%16 and
// row l/16 + 4r (f64) or row 4(l/16) + r (f32) -- both measured on gfx950.
#include <algorithm>

#include "gemm.hpp"

namespace seqx {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));

template <class T>
struct Mfma;

template <>
struct Mfma<double> {
  typedef d4 acc_t;
  typedef d2 pair_t;
  static __device__ __forceinline__ acc_t op(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};

template <>
struct Mfma<float> {
  typedef f4 acc_t;
  typedef f2 pair_t;
  static __device__ __forceinline__ acc_t op(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

// Store one accumulator element: C = alpha * acc + beta * C (+ sigma epilogue), in FP64 arithmetic.
template <class To, bool EPI>
__device__ __forceinline__ void store_elem(To* __restrict__ C, long ldc, long b, int row, int col, double alpha,
                                           double accv, double beta, const SigmaEpilogue& ep) {
  double v = alpha * accv;
  To* cp = C + static_cast<long>(row) * ldc + col;
  if (beta != 0.0) v += beta * static_cast<double>(*cp);
  if (EPI) {
    const long vo = ((b / ep.vdiv) % ep.kv) * ep.strideV + static_cast<long>(row) * ldc + col;
    v += (ep.eps[ep.nocc + col] - ep.eps[row]) * ep.V[vo];
  }
  *cp = static_cast<To>(v);
}

// ---------------------------------------------------------------- general tiles

template <class T, class To, int WM, int WN, int TM, int TN, bool TA, bool TB, bool EPI>
__global__ void __launch_bounds__(256) gemm_kernel(int M, int N, int K, double alpha, const T* __restrict__ A, long lda,
                                                   long sA, const T* __restrict__ B, long ldb, long sB, double beta,
                                                   To* __restrict__ C, long ldc, long sC, SigmaEpilogue ep) {
  typedef Mfma<T> MF;
  constexpr int BM = WM * TM * 16, BN = WN * TN * 16, BK = 16;
  __shared__ T As[BK][BM];
  __shared__ T Bs[BK][BN];
  const long b = blockIdx.z;
  A += b * sA;
  B += b * sB;
  C += b * sC;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave / WN) * TM * 16, wn = (wave % WN) * TN * 16;
  typename MF::acc_t acc[TM][TN];
  for (int i = 0; i < TM; ++i)
    for (int j = 0; j < TN; ++j) acc[i][j] = typename MF::acc_t{0, 0, 0, 0};

  for (int k0 = 0; k0 < K; k0 += BK) {
    for (int e = tid; e < BM * BK; e += 256) {
      int i, kk;
      if (!TA) { i = e / BK; kk = e % BK; } else { kk = e / BM; i = e % BM; }
      const int gi = m0 + i, gk = k0 + kk;
      T v = 0;
      if (gi < M && gk < K) v = TA ? A[static_cast<long>(gk) * lda + gi] : A[static_cast<long>(gi) * lda + gk];
      As[kk][i] = v;
    }
    for (int e = tid; e < BK * BN; e += 256) {
      int j, kk;
      if (!TB) { kk = e / BN; j = e % BN; } else { j = e / BK; kk = e % BK; }
      const int gj = n0 + j, gk = k0 + kk;
      T v = 0;
      if (gj < N && gk < K) v = TB ? B[static_cast<long>(gj) * ldb + gk] : B[static_cast<long>(gk) * ldb + gj];
      Bs[kk][j] = v;
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < BK; ks += 4) {
      T a[TM], bb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = As[ks + (lane >> 4)][wm + i * 16 + (lane & 15)];
#pragma unroll
      for (int j = 0; j < TN; ++j) bb[j] = Bs[ks + (lane >> 4)][wn + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = MF::op(a[i], bb[j], acc[i][j]);
    }
    __syncthreads();
  }

  for (int i = 0; i < TM; ++i)
    for (int j = 0; j < TN; ++j)
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm + i * 16 + MF::row(lane, r);
        const int col = n0 + wn + j * 16 + (lane & 15);
        if (row < M && col < N) store_elem<To, EPI>(C, ldc, b, row, col, alpha, acc[i][j][r], beta, ep);
      }
}

// ---------------------------------------------------------------- large tiles
// For the dense transforms: BM x BN tiles, each of the four wavefronts owns a
// BM / 2 x BN / 2 quadrant (64 x 64 of a 128 x 128 tile: 4 x 4 MFMA tiles);
// loads of element pairs.  The K panels are
// double-buffered in LDS: the loads of a later panel are issued (and kept
// ahead of the MFMAs by a scheduling barrier) before the MFMAs of the current
// one and land in the other LDS buffer afterwards, so one barrier per panel
// suffices.  Both precisions prefetch two panels ahead with two register sets
// and use buffer loads on interior tiles; FP32 also issues its LDS operand
// reads one k-step ahead of the MFMAs.  Interior and edge tiles take separate code
// paths.  Pair loads are buffer loads, which need element-aligned (dword)
// addresses only, so any leading dimension will do.  Every tile size sums an
// element in the same order: the size never changes a result.  Panel depth: 16 (FP64) or 32
// (FP32), which keeps the loads of one panel at 16 registers per lane either
// way.
constexpr int kPad = 2;

template <class T>
struct Panel {
  static constexpr int BK = sizeof(T) == 8 ? 16 : 32;
};
// element pairs per thread of a panel W rows (A) or columns (B) wide
template <class T, int W>
constexpr int kPairs = W * Panel<T>::BK / 2 / 256;

// Edge tiles and the K head panel: element loads at clamped indices, so every
// load is issued unconditionally (which keeps the wait counters exact).  Rows
// past M and columns past N only feed outputs that are never stored, so their
// clamped values are harmless; columns k >= K are set to zero.
template <class T, bool TA, bool TB, int BM, int BN>
__device__ __forceinline__ void panel_load_edge(const T* __restrict__ A, long lda, const T* __restrict__ B, long ldb,
                                                int M, int N, int K, int m0, int n0, int k0, int tid,
                                                typename Mfma<T>::pair_t* ra, typename Mfma<T>::pair_t* rb) {
  constexpr int BK = Panel<T>::BK, HK = BK / 2, HM = BM / 2, HN = BN / 2;
  auto ld_a = [&](int gi, int gk) {
    const T v = TA ? A[static_cast<long>(min(gk, K - 1)) * lda + min(gi, M - 1)]
                   : A[static_cast<long>(min(gi, M - 1)) * lda + min(gk, K - 1)];
    return gk < K ? v : T(0);
  };
  auto ld_b = [&](int gj, int gk) {
    const T v = TB ? B[static_cast<long>(min(gj, N - 1)) * ldb + min(gk, K - 1)]
                   : B[static_cast<long>(min(gk, K - 1)) * ldb + min(gj, N - 1)];
    return gk < K ? v : T(0);
  };
#pragma unroll
  for (int j = 0; j < kPairs<T, BM>; ++j) {
    const int c = tid + 256 * j;
    if (!TA) {
      const int gi = m0 + c / HK, gk = k0 + (c % HK) * 2;
      ra[j].x = ld_a(gi, gk);
      ra[j].y = ld_a(gi, gk + 1);
    } else {
      const int gk = k0 + c / HM, gi = m0 + (c % HM) * 2;
      ra[j].x = ld_a(gi, gk);
      ra[j].y = ld_a(gi + 1, gk);
    }
  }
#pragma unroll
  for (int j = 0; j < kPairs<T, BN>; ++j) {
    const int c = tid + 256 * j;
    if (!TB) {
      const int gk = k0 + c / HN, gj = n0 + (c % HN) * 2;
      rb[j].x = ld_b(gj, gk);
      rb[j].y = ld_b(gj + 1, gk);
    } else {
      const int gj = n0 + c / HK, gk = k0 + (c % HK) * 2;
      rb[j].x = ld_b(gj, gk);
      rb[j].y = ld_b(gj, gk + 1);
    }
  }
}

// Interior panels: buffer loads from a descriptor at the tile's corner, with
// the panel's position as a scalar offset and a per-thread 32-bit offset fixed
// for the whole tile, so each load needs one vector register for its address.
// Word 3 of the descriptor (0x00020000) is the gfx9 raw-buffer format.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0x7fffffff, 0x00020000);
}

template <class T>
__device__ __forceinline__ typename Mfma<T>::pair_t buffer_pair(__amdgpu_buffer_rsrc_t r, unsigned voff,
                                                                unsigned soff);
template <>
__device__ __forceinline__ f2 buffer_pair<float>(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
  return __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
template <>
__device__ __forceinline__ d2 buffer_pair<double>(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
  return __builtin_bit_cast(d2, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

template <class T, int BM, int BN>
__device__ __forceinline__ void panel_load_fast(__amdgpu_buffer_rsrc_t ar, unsigned asoff, __amdgpu_buffer_rsrc_t br,
                                                unsigned bsoff, const unsigned* oa, const unsigned* ob,
                                                typename Mfma<T>::pair_t* ra, typename Mfma<T>::pair_t* rb) {
#pragma unroll
  for (int j = 0; j < kPairs<T, BM>; ++j) ra[j] = buffer_pair<T>(ar, oa[j], asoff);
#pragma unroll
  for (int j = 0; j < kPairs<T, BN>; ++j) rb[j] = buffer_pair<T>(br, ob[j], bsoff);
}

template <class T, bool TA, bool TB, int BM, int BN>
__device__ __forceinline__ void panel_store(T (*As)[BM + kPad], T (*Bs)[BN + kPad], int tid,
                                            const typename Mfma<T>::pair_t* ra, const typename Mfma<T>::pair_t* rb) {
  constexpr int BK = Panel<T>::BK, HK = BK / 2, HM = BM / 2, HN = BN / 2;
#pragma unroll
  for (int j = 0; j < kPairs<T, BM>; ++j) {
    const int c = tid + 256 * j;
    if (!TA) {
      const int i = c / HK, kk = (c % HK) * 2;
      As[kk][i] = ra[j].x;
      As[kk + 1][i] = ra[j].y;
    } else {
      const int kk = c / HM, i = (c % HM) * 2;
      As[kk][i] = ra[j].x;
      As[kk][i + 1] = ra[j].y;
    }
  }
#pragma unroll
  for (int j = 0; j < kPairs<T, BN>; ++j) {
    const int c = tid + 256 * j;
    if (!TB) {
      const int kk = c / HN, jj = (c % HN) * 2;
      Bs[kk][jj] = rb[j].x;
      Bs[kk][jj + 1] = rb[j].y;
    } else {
      const int jj = c / HK, kk = (c % HK) * 2;
      Bs[kk][jj] = rb[j].x;
      Bs[kk + 1][jj] = rb[j].y;
    }
  }
}

// FP32: the operands of k-step s + 1 are read from LDS before the MFMAs of
// step s are issued, so the LDS latency overlaps the matrix-core work.  FP64
// keeps one operand set: its accumulators take twice the registers, and a
// second set would cost a wavefront per SIMD.
template <class T, int TM, int TN>
__device__ __forceinline__ void panel_mfma(const T (*As)[TM * 32 + kPad], const T (*Bs)[TN * 32 + kPad], int lane, int wm,
                                           int wn, typename Mfma<T>::acc_t (*acc)[TN]) {
  constexpr int NS = Panel<T>::BK / 4;
  if constexpr (sizeof(T) == 8) {  // FP64: one operand set, order left to the compiler
#pragma unroll
    for (int ks = 0; ks < Panel<T>::BK; ks += 4) {
      T a[TM], bb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = As[ks + (lane >> 4)][wm + i * 16 + (lane & 15)];
#pragma unroll
      for (int j = 0; j < TN; ++j) bb[j] = Bs[ks + (lane >> 4)][wn + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = Mfma<T>::op(a[i], bb[j], acc[i][j]);
    }
    return;
  }
  T a[2][TM], bb[2][TN];
  auto read = [&](int ks, T* ar, T* br) {
#pragma unroll
    for (int i = 0; i < TM; ++i) ar[i] = As[ks + (lane >> 4)][wm + i * 16 + (lane & 15)];
#pragma unroll
    for (int j = 0; j < TN; ++j) br[j] = Bs[ks + (lane >> 4)][wn + j * 16 + (lane & 15)];
  };
  read(0, a[0], bb[0]);
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    if (s + 1 < NS) read(4 * (s + 1), a[(s + 1) & 1], bb[(s + 1) & 1]);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = Mfma<T>::op(a[s & 1][i], bb[s & 1][j], acc[i][j]);
  }
  // schedule: the LDS reads of step 0, then per step the reads of step s + 1
  // ahead of the 4 TN MFMAs of step s (masks: 0x100 LDS read, 0x008 MFMA)
  __builtin_amdgcn_sched_group_barrier(0x100, TM + TN, 0);
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    if (s + 1 < NS) __builtin_amdgcn_sched_group_barrier(0x100, TM + TN, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0);
  }
}

// EM: 0 interior tile; 1 edge tile whose pair dimensions (M when A is
// transposed, N when B is not) are even, loaded like an interior tile at
// clamped offsets; 2 other edge tiles, element loads.
template <class T, class To, bool TA, bool TB, bool EPI, int EM, int BM, int BN>
__device__ __forceinline__ void tile_product(int M, int N, int K, double alpha, const T* __restrict__ A, long lda,
                                        const T* __restrict__ B, long ldb, double beta, To* __restrict__ C, long ldc,
                                        long b, const SigmaEpilogue& ep, int m0, int n0, T (*As)[BM + kPad],
                                        T (*Bs)[BN + kPad]) {
  typedef Mfma<T> MF;
  constexpr int BK = Panel<T>::BK, TM = BM / 32, TN = BN / 32, NPA = kPairs<T, BM>, NPB = kPairs<T, BN>;
  constexpr bool EDGE = EM != 0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);
  typename MF::acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = typename MF::acc_t{0, 0, 0, 0};
  typedef typename MF::pair_t P2;
  {
    // K is walked as a head panel of K % BK columns (when K is not a multiple
    // of BK), loaded with zero fill, followed by full panels, so that the
    // steady-state loop holds no K checks.  Two register sets for the
    // global prefetch: the loads of panel p + 2 are issued while panel p is
    // multiplied and have two panels of MFMA work to land before they are
    // stored to LDS.  The loads are unconditional (past the last panel they
    // repeat it and are not stored): a conditional load would make the wait
    // before the LDS stores cover the newest loads as well.
    P2 ra0[kPairs<T, BM>], rb0[NPB], ra1[kPairs<T, BM>], rb1[NPB];
    const int kr = K % BK;
    const int npan = K / BK + (kr ? 1 : 0);
    const int kshift = kr ? kr - BK : 0;  // panel p >= 1 starts at p * BK + kshift
    constexpr int HK = BK / 2, HM = BM / 2, HN = BN / 2;
    // Byte offsets inside a panel.  On edge tiles (EM == 1) rows and columns
    // past M and N are clamped to the last ones (pair starts to the last
    // pair): they only feed outputs that are not stored.
    const int im = M - 1 - m0, in = N - 1 - n0;  // last valid row / column of the tile
    unsigned oa[kPairs<T, BM>], ob[NPB];
#pragma unroll
    for (int j = 0; j < kPairs<T, BM>; ++j) {
      const int c = tid + 256 * j;
      int i = TA ? (c % HM) * 2 : c / HK, kk = TA ? c / HM : (c % HK) * 2;
      if (EM == 1) i = TA ? min(i, im - 1) : min(i, im);
      oa[j] = static_cast<unsigned>(TA ? kk * lda + i : i * lda + kk) * sizeof(T);
    }
#pragma unroll
    for (int j = 0; j < NPB; ++j) {
      const int c = tid + 256 * j;
      int jj = TB ? c / HK : (c % HN) * 2, kb = TB ? (c % HK) * 2 : c / HN;
      if (EM == 1) jj = TB ? min(jj, in) : min(jj, in - 1);
      ob[j] = static_cast<unsigned>(TB ? jj * ldb + kb : kb * ldb + jj) * sizeof(T);
    }
    const __amdgpu_buffer_rsrc_t ar = buffer_rsrc(TA ? A + m0 : A + static_cast<long>(m0) * lda);
    const __amdgpu_buffer_rsrc_t br = buffer_rsrc(TB ? B + static_cast<long>(n0) * ldb : B + n0);
    auto load_full = [&](int p, P2* ra, P2* rb) {
      const int k0 = p * BK + kshift;
      if (EM < 2)
        panel_load_fast<T, BM, BN>(ar, static_cast<unsigned>(TA ? k0 * lda : k0) * sizeof(T), br,
                               static_cast<unsigned>(TB ? k0 : k0 * ldb) * sizeof(T), oa, ob, ra, rb);
      else
        panel_load_edge<T, TA, TB, BM, BN>(A, lda, B, ldb, M, N, K, m0, n0, k0, tid, ra, rb);
    };
    // LDS buffers 0 and 1: rows [0, BK) and [BK, 2 BK) of As / Bs
    if (kr) panel_load_edge<T, TA, TB, BM, BN>(A, lda, B, ldb, M, N, kr, m0, n0, 0, tid, ra0, rb0);
    else load_full(0, ra0, rb0);
    load_full(min(1, npan - 1), ra1, rb1);
    panel_store<T, TA, TB, BM, BN>(As, Bs, tid, ra0, rb0);
    __syncthreads();
    int kt = 0;
    for (; kt + 1 < npan; kt += 2) {
      load_full(min(kt + 2, npan - 1), ra0, rb0);
      __builtin_amdgcn_sched_barrier(0);
      panel_mfma<T, TM, TN>(As, Bs, lane, wm, wn, acc);
      panel_store<T, TA, TB, BM, BN>(As + BK, Bs + BK, tid, ra1, rb1);
      __syncthreads();
      load_full(min(kt + 3, npan - 1), ra1, rb1);
      __builtin_amdgcn_sched_barrier(0);
      panel_mfma<T, TM, TN>(As + BK, Bs + BK, lane, wm, wn, acc);
      if (kt + 2 < npan) panel_store<T, TA, TB, BM, BN>(As, Bs, tid, ra0, rb0);
      __syncthreads();
    }
    if (kt < npan) panel_mfma<T, TM, TN>(As, Bs, lane, wm, wn, acc);  // odd panel count: the last one is in buffer 0
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm + i * 16 + MF::row(lane, r);
        const int col = n0 + wn + j * 16 + (lane & 15);
        if (!EDGE || (row < M && col < N)) store_elem<To, EPI>(C, ldc, b, row, col, alpha, acc[i][j][r], beta, ep);
      }
}

template <class T, class To, bool TA, bool TB, bool EPI, int BM, int BN>
__global__ void __launch_bounds__(256) gemm_tile_kernel(int M, int N, int K, double alpha, const T* __restrict__ A,
                                                      long lda, long sA, const T* __restrict__ B, long ldb, long sB,
                                                      double beta, To* __restrict__ C, long ldc, long sC,
                                                      SigmaEpilogue ep) {
  constexpr int BK = Panel<T>::BK;
  __shared__ T As[2 * BK][BM + kPad];
  __shared__ T Bs[2 * BK][BN + kPad];
  const long b = blockIdx.z;
  // Workgroups go to the 8 XCDs round-robin by linear id, and each XCD has its
  // own L2.  Regroup the ids so that each XCD gets a contiguous run of tiles in
  // row-major order: the column tiles of one row panel of A then share an L2
  // (the ids past the largest multiple of 8 keep their place).
  const int nbx = gridDim.x, nb = gridDim.x * gridDim.y, nfull = nb - nb % 8;
  int bid = blockIdx.y * nbx + blockIdx.x;
  if (bid < nfull) bid = (bid % 8) * (nfull / 8) + bid / 8;
  const int m0 = (bid / nbx) * BM, n0 = (bid % nbx) * BN;
  if (m0 + BM <= M && n0 + BN <= N)
    tile_product<T, To, TA, TB, EPI, 0, BM, BN>(M, N, K, alpha, A + b * sA, lda, B + b * sB, ldb, beta, C + b * sC, ldc, b, ep,
                                       m0, n0, As, Bs);
  else if ((!TA || (M & 1) == 0) && (TB || (N & 1) == 0))
    tile_product<T, To, TA, TB, EPI, 1, BM, BN>(M, N, K, alpha, A + b * sA, lda, B + b * sB, ldb, beta, C + b * sC, ldc, b, ep,
                                       m0, n0, As, Bs);
  else
    tile_product<T, To, TA, TB, EPI, 2, BM, BN>(M, N, K, alpha, A + b * sA, lda, B + b * sB, ldb, beta, C + b * sC, ldc, b, ep,
                                       m0, n0, As, Bs);
}

// ---------------------------------------------------------------- dispatch

#define SEQX_DISPATCH_T(KERNEL, ...)                                                                    \
  do {                                                                                                  \
    if (!ta && !tb) hipLaunchKernelGGL((KERNEL<__VA_ARGS__, false, false, EPI>), grid, dim3(256), 0, st, \
                                       M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, ep);  \
    else if (!ta && tb) hipLaunchKernelGGL((KERNEL<__VA_ARGS__, false, true, EPI>), grid, dim3(256), 0, \
                                           st, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, ep); \
    else if (ta && !tb) hipLaunchKernelGGL((KERNEL<__VA_ARGS__, true, false, EPI>), grid, dim3(256), 0, \
                                           st, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, ep); \
    else hipLaunchKernelGGL((KERNEL<__VA_ARGS__, true, true, EPI>), grid, dim3(256), 0, st, M, N, K,     \
                            alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, ep);                       \
  } while (0)

template <class T, class To, bool EPI, int BM, int BN>
void launch_tile(hipStream_t st, bool ta, bool tb, int M, int N, int K, double alpha, const T* A, long lda, long sA,
                 const T* B, long ldb, long sB, double beta, To* C, long ldc, long sC, int batch,
                 const SigmaEpilogue& ep) {
  dim3 grid(ceil_div(N, BN), ceil_div(M, BM), batch);
  const dim3 blk(256);
  if (!ta && !tb)
    hipLaunchKernelGGL((gemm_tile_kernel<T, To, false, false, EPI, BM, BN>), grid, blk, 0, st, M, N, K, alpha, A, lda,
                       sA, B, ldb, sB, beta, C, ldc, sC, ep);
  else if (!ta && tb)
    hipLaunchKernelGGL((gemm_tile_kernel<T, To, false, true, EPI, BM, BN>), grid, blk, 0, st, M, N, K, alpha, A, lda,
                       sA, B, ldb, sB, beta, C, ldc, sC, ep);
  else if (ta && !tb)
    hipLaunchKernelGGL((gemm_tile_kernel<T, To, true, false, EPI, BM, BN>), grid, blk, 0, st, M, N, K, alpha, A, lda,
                       sA, B, ldb, sB, beta, C, ldc, sC, ep);
  else
    hipLaunchKernelGGL((gemm_tile_kernel<T, To, true, true, EPI, BM, BN>), grid, blk, 0, st, M, N, K, alpha, A, lda,
                       sA, B, ldb, sB, beta, C, ldc, sC, ep);
}

// Tile size: 128 rows by 128 columns, or 96 where that pads N by at least 3 %
// less (N = 660: 672 columns instead of 768), one workgroup per compute unit.
// 64 x 64 tiles, four workgroups per compute unit, where the padding and the
// last round of the large ones waste more than the small ones' lower rate (47
// against 63 TFLOP/s): 10040 x 502 x 251 as 316 large tiles took 80 us.
// 32 x 32 where even those leave compute units without work: one product of
// 502 rows went 71 -> 13 us, the 20 products of C100H102 (odd row
// lengths, formerly element loads in 64 x 64 tiles) 541 -> 346 us.
constexpr long kComputeUnits = 256;

template <class T, class To, bool EPI>
void launch_tiles(hipStream_t st, bool ta, bool tb, int M, int N, int K, double alpha, const T* A, long lda, long sA,
                  const T* B, long ldb, long sB, double beta, To* C, long ldc, long sC, int batch,
                  const SigmaEpilogue& ep) {
  auto padded = [](long x, long t) { return static_cast<double>(ceil_div(x, t) * t); };
  auto groups = [&](long bm, long bn) { return static_cast<long>(ceil_div(M, bm) * ceil_div(N, bn)) * batch; };
  const bool n96 = 100.0 * padded(N, 96) < 97.0 * padded(N, 128);
  const long bn = n96 ? 96 : 128, large = groups(128, bn);
  // share of the occupied compute-unit time that forms stored elements
  const double work = static_cast<double>(M) * N;
  const double use128 = work / (padded(M, 128) * padded(N, bn)) * large / padded(large, kComputeUnits);
  const double use64 = work / (padded(M, 64) * padded(N, 64));
#define SEQX_TILE(BM_, BN_)                                                                                        \
  launch_tile<T, To, EPI, BM_, BN_>(st, ta, tb, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, ep)
  if (large >= kComputeUnits && use128 >= 0.72 * use64) {
    if (n96) SEQX_TILE(128, 96);
    else SEQX_TILE(128, 128);
  } else if (groups(64, 64) >= kComputeUnits) {
    SEQX_TILE(64, 64);
  } else {
    SEQX_TILE(32, 32);
  }
#undef SEQX_TILE
}

template <class T, class To, int WM, int WN, int TM, int TN, bool EPI>
void launch_cfg(hipStream_t st, bool ta, bool tb, int M, int N, int K, double alpha, const T* A, long lda, long sA,
                const T* B, long ldb, long sB, double beta, To* C, long ldc, long sC, int batch,
                const SigmaEpilogue& ep) {
  constexpr int BM = WM * TM * 16, BN = WN * TN * 16;
  dim3 grid(ceil_div(N, BN), ceil_div(M, BM), batch);
  SEQX_DISPATCH_T(gemm_kernel, T, To, WM, WN, TM, TN);
}

template <class T, class To>
void gemm_any(hipStream_t st, bool ta, bool tb, int M, int N, int K, double alpha, const T* A, long lda, long sA,
              const T* B, long ldb, long sB, double beta, To* C, long ldc, long sC, int batch,
              const SigmaEpilogue* epi) {
  if (M <= 0 || N <= 0 || batch <= 0) return;
  if (K <= 0) {
    // an empty product: C = beta * C (only used with beta = 0 in practice)
    if (beta == 0.0)
      for (int b = 0; b < batch; ++b)
        for (int i = 0; i < M; ++i)
          SEQX_HIP(hipMemsetAsync(C + b * sC + static_cast<long>(i) * ldc, 0, N * sizeof(To), st));
    return;
  }
  SigmaEpilogue ep;
  if (epi) ep = *epi;
  if constexpr (sizeof(T) == 8 && sizeof(To) == 8) {
    if (!ta && !tb && !epi && batch == 1 && N >= 4096 && (M <= 48 || (M <= 256 && N >= 64L * M))) {
      // combinations of a long basis: passes of at most 48 output rows, each
      // reading B once
      for (int r0 = 0; r0 < M; r0 += 48)
        skinny_combine(st, std::min(48, M - r0), N, K, alpha, A + static_cast<long>(r0) * lda, lda, B, ldb, beta,
                       C + static_cast<long>(r0) * ldc, ldc);
      return;
    }
  }
  const bool skinny = N <= 16;
  // the large tiles address each operand with 32-bit byte offsets from a
  // tile corner: rows and panel steps must stay below 2 GiB
  const long ldmax = lda > ldb ? lda : ldb;
  const bool small_offsets = (ldmax * (static_cast<long>(K > 128 ? K : 128) + 128) + K) * static_cast<long>(sizeof(T)) <
                             (1L << 31);
  const bool tiles = small_offsets && M >= 32 && N >= 32 && K >= 32;
  if constexpr (sizeof(To) == 8) {  // the epilogue's products are FP64
    if (epi) {
      if (tiles)
        launch_tiles<T, To, true>(st, ta, tb, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, ep);
      else
        launch_cfg<T, To, 2, 2, 2, 2, true>(st, ta, tb, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC,
                                            batch, ep);
      SEQX_LAUNCH_CHECK();
      return;
    }
  }
  if (tiles) {
    launch_tiles<T, To, false>(st, ta, tb, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, ep);
  } else if (!skinny && M <= 32) {
    launch_cfg<T, To, 1, 4, 2, 1, false>(st, ta, tb, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch,
                                         ep);
  } else if (skinny) {
    launch_cfg<T, To, 4, 1, 1, 1, false>(st, ta, tb, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch,
                                         ep);
  } else {
    launch_cfg<T, To, 2, 2, 2, 2, false>(st, ta, tb, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch,
                                         ep);
  }
  SEQX_LAUNCH_CHECK();
}

}  // namespace

void dgemm(hipStream_t st, bool ta, bool tb, int M, int N, int K, double alpha, const double* A, long lda, long sA,
           const double* B, long ldb, long sB, double beta, double* C, long ldc, long sC, int batch,
           const SigmaEpilogue* epi) {
  gemm_any<double, double>(st, ta, tb, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, epi);
}

void sgemm(hipStream_t st, bool ta, bool tb, int M, int N, int K, double alpha, const float* A, long lda, long sA,
           const float* B, long ldb, long sB, double beta, float* C, long ldc, long sC, int batch) {
  gemm_any<float, float>(st, ta, tb, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, nullptr);
}

void sgemm_out64(hipStream_t st, bool ta, bool tb, int M, int N, int K, double alpha, const float* A, long lda,
                 long sA, const float* B, long ldb, long sB, double beta, double* C, long ldc, long sC, int batch,
                 const SigmaEpilogue* epi) {
  gemm_any<float, double>(st, ta, tb, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, epi);
}

void dgemm_cm(hipStream_t st, bool ta, bool tb, int M, int N, int K, double alpha, const double* A, long lda,
              const double* B, long ldb, double beta, double* C, long ldc) {
  // column-major C = op(A) op(B) is row-major C^T = op(B)^T op(A)^T
  dgemm(st, tb, ta, N, M, K, alpha, B, ldb, 0, A, lda, 0, beta, C, ldc, 0, 1, nullptr);
}

}  // namespace seqx
