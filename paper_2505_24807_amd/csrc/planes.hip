// Products of matrices held as bfloat16 planes (planes.hpp) on the bfloat16
// matrix cores (v_mfma_f32_16x16x32_bf16), FP32 accumulation.
#include "planes.hpp"

namespace seqx {

namespace {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- splitting

// 32 x 32 tiles through LDS: read along the source rows, write one 32-k block
// of a plane row (all its planes, 64 bytes each) per source column.
template <int NP, class T>
__global__ void __launch_bounds__(256) split_transposed_kernel(int rows, int cols, const T* __restrict__ src,
                                                               long lds, long ss, plane_t* __restrict__ dst,
                                                               long ld) {
  __shared__ float tile[32][33];
  const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
  const T* s = src + blockIdx.z * ss;
  const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = r0 + y + 8 * j, c = c0 + x;
    tile[y + 8 * j][x] = (r < rows && c < cols) ? static_cast<float>(s[static_cast<long>(r) * lds + c]) : 0.0f;
  }
  __syncthreads();
  // thread: source column c0 + t / 8, four consecutive k
  const int c = threadIdx.x >> 3, k = (threadIdx.x & 7) * 4;
  if (c0 + c >= cols) return;
  const PlaneOut<NP> out{dst, 0, ld};
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = tile[k + e][c];
  out.put4(static_cast<long>(blockIdx.z) * cols + c0 + c, r0 + k, v);
}

__global__ void __launch_bounds__(256) split_rows_kernel(int rows, int cols, const float* __restrict__ src, long lds,
                                                         plane_t* __restrict__ dst, long ld) {
  const int q = blockIdx.x * 256 + threadIdx.x;  // group of four columns
  const int r = blockIdx.y;
  if (4 * q >= cols) return;
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = 4 * q + e < cols ? src[static_cast<long>(r) * lds + 4 * q + e] : 0.0f;
  PlaneOut<3>{dst, 0, ld}.put4(r, 4 * q, v);
}

// ---------------------------------------------------------------- products

struct NoEpilogue {};

// Output of four consecutive i (i0 .. i0 + 3) of row j.
template <int NP>
__device__ __forceinline__ void store4(const PlaneOut<NP>& o, const NoEpilogue&, long, int i0, int j, int I, f4 v) {
  if (i0 >= I) return;  // past I inside the last block: masked by the reader
  float x[4] = {v[0], v[1], v[2], v[3]};
  o.put4(j, i0, x);
}
__device__ __forceinline__ void store4(const MatOut<float>& o, const NoEpilogue&, long, int i0, int j, int I, f4 v) {
  float* q = o.p + static_cast<long>(j) * o.n + i0;
  if (i0 + 3 < I) {
    __builtin_memcpy(q, &v, 16);  // element-aligned
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (i0 + e < I) q[e] = v[e];
  }
}
template <class To>
__device__ __forceinline__ void store4(const MatOut<To>& o, const SigmaEpilogue& ep, long b, int i0, int j, int I,
                                       f4 v) {
  To* q = o.p + static_cast<long>(j) * o.n + i0;
  const long vo = ((b / ep.vdiv) % ep.kv) * ep.strideV + static_cast<long>(j) * o.n + i0;
  const double ej = ep.eps[j];
  if (i0 + 3 < I) {  // whole groups: element-aligned wide loads and stores
    double vv[4], ea[4];
    To x[4];
    if (ep.Vf) {
      float vf[4];
      __builtin_memcpy(vf, ep.Vf + vo, sizeof(vf));
#pragma unroll
      for (int e = 0; e < 4; ++e) vv[e] = static_cast<double>(vf[e]);
    } else {
      __builtin_memcpy(vv, ep.V + vo, sizeof(vv));
    }
    __builtin_memcpy(ea, ep.eps + ep.nocc + i0, sizeof(ea));
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = static_cast<To>(static_cast<double>(v[e]) + (ea[e] - ej) * vv[e]);
    __builtin_memcpy(q, x, sizeof(x));
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (i0 + e < I) {
      const double vv = ep.Vf ? static_cast<double>(ep.Vf[vo + e]) : ep.V[vo + e];
      q[e] = static_cast<To>(static_cast<double>(v[e]) + (ep.eps[ep.nocc + i0 + e] - ej) * vv);
    }
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const plane_t* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<plane_t*>(base), 0, 0x7fffffff, 0x00020000);
}

// zero the elements k >= valid of one 8-element chunk that starts at k0
__device__ __forceinline__ u4 mask_chunk(u4 x, int left) {
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    if (2 * d >= left) x[d] = 0u;
    else if (2 * d + 1 >= left) x[d] &= 0xffffu;
  }
  return x;
}

constexpr int kFlush = 4;  // panels

// One BP x BQ tile: four wavefronts (2 x 2), each (BP / 2) x (BQ / 2), K in
// panels of 32.  A panel of either operand is NP planes of 16-byte chunks (8
// k); the loads of panel p + 1 go to registers while panel p is multiplied out
// of LDS.  One LDS copy (48 KB for 128 x 128 and three planes) leaves room for
// two workgroups per CU, whose matrix-core and staging phases overlap.  In LDS
// chunk c of row r sits at place c ^ ((r >> 1) & 3) of its row, so that the 8
// lanes of one LDS cycle (8 rows, one chunk each) touch all banks once.
// SP, SQ: planes stored in P and Q (the first NP are used).
//
// Six products a value: 145-165 TFLOP/s of FP32 work or 0.9-1.0 PFLOP/s in
// bfloat16 (a large library bfloat16 product reaches 1.1 on this card; the FP32
// matrix cores gave 93-115).  Counters of the four products of (H2O)330, 32
// vectors: matrix cores busy 50-58 % of the cycles, LDS 39-43 % (a quarter of it
// bank conflicts), memory at most 3.6 TB/s, and a clock of 1.7 GHz where the FP64
// products run at 2.3: no unit is full, the clock and the staging of a panel that
// two workgroups overlap only in part set the time.  (H2O)330, 20
// vectors, TDHF: C_o V 0.62 -> 0.43 ms, T1 C_v^T 0.97 -> 0.60, F C_v 1.80 ->
// 1.29, C_o^T Z 1.49 -> 1.10; the whole products 5.23 -> 3.87 ms, with the
// error against FP64 9.3e-8 -> 3.3e-8.  Two planes, (H2O)200, 32 vectors:
// 1.55 -> 1.27 ms against splitting in the product kernel.  Measured slower:
// 256 x 96 and 256 x 128 tiles of 8 wavefronts with two LDS copies (C_o V
// 0.52 ms), and second accumulators (230 registers, one workgroup per CU less).
template <int NP, int SP, int SQ, int BP, int BQ, class Out, class Epi>
__global__ void __launch_bounds__(256, 2) plane_gemm_kernel(int I, int J, int K, const plane_t* __restrict__ P,
                                                            long sP, const plane_t* __restrict__ Q, long sQ, Out out,
                                                            Epi ep) {
  constexpr int TP = BP / 32, TQ = BQ / 32;
  constexpr int RC = NP * 4;                                    // chunks per row and panel
  constexpr int LP = (BP * RC + 255) / 256, LQ = (BQ * RC + 255) / 256;  // chunks per thread
  __shared__ u4 Ls[(BP + BQ) * RC];
  u4* Lp = Ls;
  u4* Lq = Ls + BP * RC;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // Workgroup ids go round-robin over the 8 XCDs, each with its own L2.  The
  // tiles of the whole stack are dealt out in contiguous runs per XCD with the
  // shorter of I and J fastest: a run sweeps the smaller operand, which L2
  // keeps best, against one row panel of the larger one.
  const int ni = (I + BP - 1) / BP, nj = (J + BQ - 1) / BQ;
  const unsigned ntot = gridDim.x, nfull = ntot - ntot % 8;
  unsigned id = blockIdx.x;
  if (id < nfull) id = (id % 8) * (nfull / 8) + id / 8;
  const long b = id / (ni * nj);
  const int t = id % (ni * nj);
  const bool ifast = I <= J;
  const int i0 = (ifast ? t % ni : t / nj) * BP, j0 = (ifast ? t / ni : t % nj) * BQ;
  const int kb = (K + kPlaneK - 1) / kPlaneK;
  const long pp = static_cast<long>(kb) * SP * kPlaneK, pq = static_cast<long>(kb) * SQ * kPlaneK;
  const __amdgpu_buffer_rsrc_t rp = row_rsrc(P + b * sP + i0 * pp), rq = row_rsrc(Q + b * sQ + j0 * pq);
  // byte offsets of this thread's chunks inside panel 0; rows past I or J are
  // clamped (they only feed outputs that are not stored)
  unsigned op[LP], oq[LQ];
#pragma unroll
  for (int j = 0; j < LP; ++j) {
    const int c = min(tid + 256 * j, BP * RC - 1), r = min(c / RC, I - 1 - i0);
    op[j] = static_cast<unsigned>(r * pp * 2) + (c % RC) * 16;
  }
#pragma unroll
  for (int j = 0; j < LQ; ++j) {
    const int c = min(tid + 256 * j, BQ * RC - 1), r = min(c / RC, J - 1 - j0);
    oq[j] = static_cast<unsigned>(r * pq * 2) + (c % RC) * 16;
  }
  u4 gp[LP], gq[LQ];
  auto load = [&](int p) {
#pragma unroll
    for (int j = 0; j < LP; ++j)
      gp[j] = __builtin_bit_cast(u4, __builtin_amdgcn_raw_buffer_load_b128(rp, op[j], p * (SP * 64), 0));
#pragma unroll
    for (int j = 0; j < LQ; ++j)
      gq[j] = __builtin_bit_cast(u4, __builtin_amdgcn_raw_buffer_load_b128(rq, oq[j], p * (SQ * 64), 0));
  };
  auto place = [&](int c, int rows) {  // LDS unit of chunk c: [plane][row][swizzled chunk]
    const int r = c / RC, pl = (c % RC) / 4, kc = c % 4;
    return (pl * rows + r) * 4 + (kc ^ ((r >> 1) & 3));
  };
  auto store = [&](bool last) {
#pragma unroll
    for (int j = 0; j < LP; ++j) {
      const int c = tid + 256 * j;
      u4 x = gp[j];
      if (last) x = mask_chunk(x, K - (kb - 1) * kPlaneK - (c % 4) * 8);
      if (BP * RC % 256 == 0 || c < BP * RC) Lp[place(c, BP)] = x;
    }
#pragma unroll
    for (int j = 0; j < LQ; ++j) {
      const int c = tid + 256 * j;
      u4 x = gq[j];
      if (last) x = mask_chunk(x, K - (kb - 1) * kPlaneK - (c % 4) * 8);
      if (BQ * RC % 256 == 0 || c < BQ * RC) Lq[place(c, BQ)] = x;
    }
  };
  const int wp = (wave >> 1) * (BP / 2), wq = (wave & 1) * (BQ / 2);
  const int r = lane & 15, sw = (lane >> 4) ^ ((r >> 1) & 3);
  f4 acc[TP][TQ];
#pragma unroll
  for (int i = 0; i < TP; ++i)
#pragma unroll
    for (int j = 0; j < TQ; ++j) acc[i][j] = f4{0, 0, 0, 0};
  auto multiply = [&]() {
    bf8 a[NP][TP], c[NP][TQ];
#pragma unroll
    for (int q = 0; q < NP; ++q) {
#pragma unroll
      for (int i = 0; i < TP; ++i)
        a[q][i] = __builtin_bit_cast(bf8, Lp[(q * BP + wp + 16 * i + r) * 4 + sw]);
#pragma unroll
      for (int j = 0; j < TQ; ++j)
        c[q][j] = __builtin_bit_cast(bf8, Lq[(q * BQ + wq + 16 * j + r) * 4 + sw]);
    }
    auto mma = [&](int qa, int qc) {
#pragma unroll
      for (int i = 0; i < TP; ++i)
#pragma unroll
        for (int j = 0; j < TQ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[qa][i], c[qc][j], acc[i][j], 0, 0, 0);
    };
    if constexpr (NP == 3) {  // smallest products first
      mma(2, 0);
      mma(0, 2);
      mma(1, 1);
    }
    mma(1, 0);
    mma(0, 1);
    mma(0, 0);
  };
  f4 sum[TP][TQ];
  if constexpr (NP == 3)
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < TQ; ++j) sum[i][j] = f4{0, 0, 0, 0};
  // three planes: the running products go into the sums every kFlush panels,
  // so that most roundings happen at the size of a partial sum
  auto flush = [&]() {
    if constexpr (NP == 3)
#pragma unroll
      for (int i = 0; i < TP; ++i)
#pragma unroll
        for (int j = 0; j < TQ; ++j) {
          sum[i][j] += acc[i][j];
          acc[i][j] = f4{0, 0, 0, 0};
        }
  };
  load(0);
  for (int p = 0; p + 1 < kb; ++p) {
    store(false);
    __syncthreads();
    load(p + 1);
    multiply();
    if (p % kFlush == kFlush - 1) flush();
    __syncthreads();
  }
  store(true);
  __syncthreads();
  multiply();
  if constexpr (NP == 3)
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < TQ; ++j) acc[i][j] += sum[i][j];
  const Out o = out.at(b);
#pragma unroll
  for (int i = 0; i < TP; ++i)
#pragma unroll
    for (int j = 0; j < TQ; ++j) {
      const int jj = j0 + wq + 16 * j + r;
      if (jj < J) store4(o, ep, b, i0 + wp + 16 * i + 4 * (lane >> 4), jj, I, acc[i][j]);
    }
}

// Tile choice: 128 x 128; 96 along the dimension that it pads at least 3 %
// less (v = 660: 672 instead of 768); 64 x 64 when the large tiles would leave
// compute units idle (fewer than two workgroups each).
constexpr int kFewTiles = 512;

bool pads_less_96(int n) {
  const long w128 = static_cast<long>(ceil_div(n, 128)) * 128, w96 = static_cast<long>(ceil_div(n, 96)) * 96;
  return 100 * w96 < 97 * w128;
}

template <int NP, int SP, int SQ, int BP, int BQ, class Out, class Epi>
void launch_tile(hipStream_t st, const PlaneGemm& g, const Out& out, const Epi& ep) {
  const dim3 grid(ceil_div(g.I, BP) * ceil_div(g.J, BQ) * g.batch);
  hipLaunchKernelGGL((plane_gemm_kernel<NP, SP, SQ, BP, BQ, Out, Epi>), grid, dim3(256), 0, st, g.I, g.J, g.K, g.P,
                     g.sP, g.Q, g.sQ, out, ep);
  SEQX_LAUNCH_CHECK();
}

// W96: 96 along I (1), along J (2) or not at all (0)
template <int NP, int SP, int SQ, int W96, class Out, class Epi>
void launch(hipStream_t st, const PlaneGemm& g, const Out& out, const Epi& ep) {
  if (g.I <= 0 || g.J <= 0 || g.K <= 0 || g.batch <= 0) return;
  const long tiles = static_cast<long>(ceil_div(g.I, 128)) * ceil_div(g.J, 128) * g.batch;
  if (tiles < kFewTiles) {
    launch_tile<NP, SP, SQ, 64, 64>(st, g, out, ep);
    return;
  }
  if constexpr (W96 == 1) {
    if (pads_less_96(g.I)) {
      launch_tile<NP, SP, SQ, 96, 128>(st, g, out, ep);
      return;
    }
  }
  if constexpr (W96 == 2) {
    if (pads_less_96(g.J)) {
      launch_tile<NP, SP, SQ, 128, 96>(st, g, out, ep);
      return;
    }
  }
  launch_tile<NP, SP, SQ, 128, 128>(st, g, out, ep);
}

}  // namespace

template <class T>
void split_transposed(hipStream_t st, int planes, int batch, int rows, int cols, const T* src, long lds, long ss,
                      plane_t* dst) {
  const dim3 grid(ceil_div(cols, 32), ceil_div(rows, 32), batch);
  const long ld = plane_row(rows, planes);
  if (planes == 3)
    hipLaunchKernelGGL((split_transposed_kernel<3, T>), grid, dim3(256), 0, st, rows, cols, src, lds, ss, dst, ld);
  else
    hipLaunchKernelGGL((split_transposed_kernel<2, T>), grid, dim3(256), 0, st, rows, cols, src, lds, ss, dst, ld);
  SEQX_LAUNCH_CHECK();
}
template void split_transposed<float>(hipStream_t, int, int, int, int, const float*, long, long, plane_t*);
template void split_transposed<double>(hipStream_t, int, int, int, int, const double*, long, long, plane_t*);

void split_rows(hipStream_t st, int rows, int cols, const float* src, long lds, plane_t* dst) {
  hipLaunchKernelGGL(split_rows_kernel, dim3(ceil_div(cols, 1024), rows), dim3(256), 0, st, rows, cols, src, lds, dst,
                     plane_row(cols, 3));
  SEQX_LAUNCH_CHECK();
}

void plane_gemm_planes(hipStream_t st, const PlaneGemm& g, plane_t* out, long sO) {
  const NoEpilogue ep;
  // T1 (K = o, I = v) tiles 96 along I; Z^T (I = n, J = v) along J
  if (g.planes == 3) {
    const PlaneOut<3> o{out, sO, plane_row(g.I, 3)};
    if (g.J < g.I) launch<3, 3, 3, 2>(st, g, o, ep);
    else launch<3, 3, 3, 1>(st, g, o, ep);
  } else {
    const PlaneOut<2> o{out, sO, plane_row(g.I, 2)};
    if (g.J < g.I) launch<2, 2, 3, 2>(st, g, o, ep);
    else launch<2, 2, 3, 1>(st, g, o, ep);
  }
}

void plane_gemm_f32(hipStream_t st, const PlaneGemm& g, float* out, long ldo) {
  const MatOut<float> o{out, 0, static_cast<int>(ldo)};
  if (g.planes == 3) launch<3, 3, 3, 0>(st, g, o, NoEpilogue{});
  else launch<2, 3, 2, 0>(st, g, o, NoEpilogue{});
}

template <class To>
void plane_gemm_sigma(hipStream_t st, const PlaneGemm& g, To* out, long ldo, long sO, const SigmaEpilogue& ep) {
  const MatOut<To> o{out, sO, static_cast<int>(ldo)};
  if (g.planes == 3) launch<3, 3, 3, 1>(st, g, o, ep);
  else launch<2, 2, 3, 1>(st, g, o, ep);
}
template void plane_gemm_sigma<float>(hipStream_t, const PlaneGemm&, float*, long, long, const SigmaEpilogue&);
template void plane_gemm_sigma<double>(hipStream_t, const PlaneGemm&, double*, long, long, const SigmaEpilogue&);

}  // namespace seqx
