// FP32 matrices as bfloat16 planes, and their products on the bfloat16 matrix
// cores (low-precision transforms of the sigma build).
//
// A value x is kept as hi = bf16(x), mid = bf16(x - hi), lo = x - hi - mid
// (round to nearest even): 8 + 8 + 8 significant bits hold the 24 bits of an
// FP32 value exactly.  Two planes (hi, mid) are the split-bfloat16 form.
//
// Layout ("plane rows"): a matrix row of length K is ceil(K / 32) blocks; a
// block holds its planes one after another, 32 consecutive k each (64 bytes a
// plane).  Every operand has the summation index along its rows, so a panel of
// 32 k is one contiguous piece per row and reaches the matrix-core operand
// layout without any conversion or transposition.  Positions past K hold
// anything: the product kernels mask them.
#pragma once

#include "common.hpp"
#include "gemm.hpp"

namespace seqx {

typedef unsigned short plane_t;  // bfloat16 bits

constexpr int kPlaneK = 32;  // k per block

inline long plane_blocks(int K) { return (K + kPlaneK - 1) / kPlaneK; }
// elements of one plane row
inline long plane_row(int K, int planes) { return plane_blocks(K) * planes * kPlaneK; }

// hi, mid, lo of one value.  A finite value whose hi would round to infinity
// is truncated instead; non-finite values keep their hi and zeros.
__device__ __forceinline__ void split_planes(float x, __bf16& hi, __bf16& mid, __bf16& lo) {
  hi = static_cast<__bf16>(x);
  float r = x - static_cast<float>(hi);
  if (!(__builtin_fabsf(r) < __builtin_inff())) {
    if (__builtin_fabsf(x) < __builtin_inff()) {
      const float t = __uint_as_float(__float_as_uint(x) & 0xffff0000u);
      hi = static_cast<__bf16>(t);
      r = x - t;
    } else {
      r = 0.0f;
    }
  }
  mid = static_cast<__bf16>(r);
  lo = static_cast<__bf16>(r - static_cast<float>(mid));
}

// Destination of matrix elements as plane rows with NP planes: `p` the matrix,
// `s` elements between matrices of a stack, `ld` elements per row.
template <int NP>
struct PlaneOut {
  typedef float stage_t;  // type of staged elements (what the planes represent)
  plane_t* p;
  long s, ld;
  __device__ __forceinline__ PlaneOut at(long i) const { return {p + i * s, s, ld}; }
  __device__ __forceinline__ plane_t* pos(long row, int col) const {
    return p + row * ld + static_cast<long>(col >> 5) * (NP * kPlaneK) + (col & 31);
  }
  __device__ __forceinline__ void put(long row, int col, double v) const {
    plane_t* q = pos(row, col);
    __bf16 h[3];
    split_planes(static_cast<float>(v), h[0], h[1], h[2]);
#pragma unroll
    for (int k = 0; k < NP; ++k) q[k * kPlaneK] = __builtin_bit_cast(plane_t, h[k]);
  }
  // four consecutive columns, col a multiple of 4
  __device__ __forceinline__ void put4(long row, int col, const float* v) const {
    typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
    plane_t* q = pos(row, col);
    bf4 h[3];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      __bf16 a, b, c;
      split_planes(v[e], a, b, c);
      h[0][e] = a;
      h[1][e] = b;
      h[2][e] = c;
    }
#pragma unroll
    for (int k = 0; k < NP; ++k) *reinterpret_cast<bf4*>(q + k * kPlaneK) = h[k];
  }
};

// Destination of matrix elements stored as they are: row-major, leading dimension n.
template <class T>
struct MatOut {
  typedef T stage_t;
  T* p;
  long s;
  int n;
  __device__ __forceinline__ MatOut at(long i) const { return {p + i * s, s, n}; }
  __device__ __forceinline__ void put(long row, int col, double v) const { p[row * n + col] = static_cast<T>(v); }
};

// dst (stack of `batch` matrices, cols x rows as three-plane or two-plane rows,
// row length `rows`) = transpose of src (rows x cols, leading dimension lds,
// matrices ss apart).  FP64 sources are rounded to FP32 first.
template <class T>
void split_transposed(hipStream_t st, int planes, int batch, int rows, int cols, const T* src, long lds, long ss,
                      plane_t* dst);
// dst (rows x cols as three-plane rows) = src
void split_rows(hipStream_t st, int rows, int cols, const float* src, long lds, plane_t* dst);

// Products out[j][i] = sum_k P[i][k] Q[j][k] over stacks of matrices, P (I
// rows) and Q (J rows) plane rows of K values.  `planes` = 3: six bfloat16
// products of the exact splits (hi hi, hi mid, mid hi, mid mid, hi lo, lo hi;
// the dropped ones are below 2^-24 of |x||y|) with FP32 accumulation, which
// measures closer to FP64 than the FP32 matrix cores; 2: hi hi, hi mid, mid hi.
// The orbital operand always has three stored planes, the other one `planes`.
struct PlaneGemm {
  int planes, batch, I, J, K;
  const plane_t *P, *Q;
  long sP, sQ;  // elements between the matrices of a stack (0: shared)
};
// orbitals in Q, output as plane rows (row length I): T1 = C_o V, Z^T = C_v^T F^T
void plane_gemm_planes(hipStream_t st, const PlaneGemm& g, plane_t* out, long sO);
// orbitals in P, FP32 output: R = T1 C_v^T
void plane_gemm_f32(hipStream_t st, const PlaneGemm& g, float* out, long ldo);
// orbitals in Q, FP32 or FP64 output plus the (eps_a - eps_i) V term: C_o^T Z + de V
template <class To>
void plane_gemm_sigma(hipStream_t st, const PlaneGemm& g, To* out, long ldo, long sO, const SigmaEpilogue& ep);

}  // namespace seqx
