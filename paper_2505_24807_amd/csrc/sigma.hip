// Matrix-free products of Eqs. 8-9 (paper, GPU-implementation subsection).
//
//   R_I   = C_o V_I C_v^T                     two MFMA GEMMs (n x o x v, n x v x n)
//   F_I   = G(R_I)                            NDDO contraction (fock.hip)
//   out_I = C_o^T F_I C_v + de o V_I          two MFMA GEMMs, de added in the epilogue
// Singlet CIS:  F = 2 J(R) - K(R).  TDHF:  (A+B) <-> 4 J(S) - 2 K(S) and
// (A-B) <-> -2 K(D) with S, D the symmetric / antisymmetric parts of R: A V
// pairs with K(R) and B V with K(R^T), which gives exactly these combinations.
#include <mutex>

#include "gemm.hpp"
#include "linalg.hpp"
#include "planes.hpp"
#include "sigma.hpp"

namespace seqx {

void PhaseTimer::reset() {
  resolve();
  for (int p = 0; p < kNumPhases; ++p) {
    ms[p] = flops[p] = bytes[p] = 0.0;
    launches[p] = 0;
  }
}

void PhaseTimer::resolve() {
  for (size_t c = 0; c < pending.size(); ++c) {
    auto& ev = pending[c];
    SEQX_HIP(hipEventSynchronize(ev[kNumPhases]));
    for (int p = 0; p < kNumPhases; ++p) {
      float t = 0.f;
      SEQX_HIP(hipEventElapsedTime(&t, ev[p], ev[p + 1]));
      ms[p] += t;
      flops[p] += pending_flops[c][p];
      bytes[p] += pending_bytes[c][p];
      launches[p] += pending_launches[c][p];
    }
    for (auto& e : ev) (void)hipEventDestroy(e);
  }
  pending.clear();
  pending_flops.clear();
  pending_bytes.clear();
  pending_launches.clear();
}

PhaseTimer::~PhaseTimer() {
  for (auto& ev : pending)
    for (auto& e : ev) (void)hipEventDestroy(e);
}

void forward_transform(const DeviceMolecule& m, int k, const double* X, double* T, SigmaWork& w, hipStream_t st) {
  const int n = m.nao, o = m.nocc, v = m.nvirt;
  w.buf.ensure(static_cast<size_t>(k) * n * v * sizeof(double));
  double* T1 = reinterpret_cast<double*>(w.buf.p);
  // T1_I (n x v) = C[:, :o] (n x o, ld n) * X_I (o x v)
  dgemm(st, false, false, n, v, o, 1.0, m.C.p, n, 0, X, v, static_cast<long>(o) * v, 0.0, T1, v,
        static_cast<long>(n) * v, k);
  // T_I (n x n) = T1_I * C[:, o:]^T, one GEMM over the stacked T1_I
  dgemm(st, false, true, k * n, n, v, 1.0, T1, v, 0, m.C.p + o, n, 0, 0.0, T, n, 0, 1);
}

namespace {

// Intermediates of one chunk of kc trial vectors: the FP64 set (T1, R, F, Z),
// the FP32 set (V32, T1s, Rs, Fs, Zs) or the plane set (Vp, T1p, Rs, Fp, Zp),
// and the contraction's work arrays.
struct ChunkBufs {
  double *T1 = nullptr, *R = nullptr, *F = nullptr, *Z = nullptr;
  float *V32 = nullptr, *T1s = nullptr, *Rs = nullptr, *Fs = nullptr, *Zs = nullptr;
  plane_t *Vp = nullptr, *T1p = nullptr, *Fp = nullptr, *Zp = nullptr;
  double *gr = nullptr, *gJ = nullptr, *gws = nullptr;
};

// FP32 trial vectors in and FP32 products out (plane transforms only), in place
// of the FP64 ones
struct F32Io {
  const float* V = nullptr;
  float* out1 = nullptr;
  float* out2 = nullptr;
};

bool has_planes(const DeviceMolecule& m, int precision) { return precision != kPrecFP64 && m.Cop.n > 0; }

// Planes of the low-precision transforms.  Split bfloat16 takes two from 96
// occupied and 96 virtual orbitals on (even numbers of both); below, and for
// odd numbers, its callers have always had FP32 accuracy, and the third plane
// costs little there (the products are bound by launches and tile remainders).
int plane_count(const DeviceMolecule& m, int precision) {
  const bool two = precision == kPrecBF16x3 && m.nocc >= 96 && m.nvirt >= 96 && m.nocc % 2 == 0 && m.nvirt % 2 == 0;
  return two ? 2 : 3;
}

// Where a chunk is formed from FP32 matrices although the molecule has planes:
// TDHF products of many vectors below 150 AOs.  The exchange kernel has a
// handful of workgroups there, each walking all vectors, and writing planes costs
// it 6.3 us a vector.  Planes are the closer to FP64 (3.8e-8 against 6.7e-8 of the
// product), so they give way only where they are slower than FP32 products have
// been without them: at 96 AOs from 16 vectors on (32 vectors: 262 us against
// 219), at 120 from 24 (279 against 253), at 144 from 28 (276 against 269); at 156
// AOs 279 against 285.  In those cases matrices now take 153, 169 and 166 us.
// CIS forms one matrix a vector and gained throughout.
bool prefers_matrices(const DeviceMolecule& m, int theory, int kc) {
  return theory == 1 && m.nao < 150 && 11 * kc > 2 * m.nao;
}

// One chunk of the product: kc vectors Vc -> out1c (and out2c), outputs os
// elements apart.  ev (optional) receives the phase boundaries.
void sigma_chunk(const DeviceMolecule& m, int theory, int kc, const double* Vc, double* out1c, double* out2c, long os,
                 int precision, const ChunkBufs& b, hipStream_t st, std::array<hipEvent_t, kNumPhases + 1>* ev,
                 const F32Io* io = nullptr) {
  const int n = m.nao, o = m.nocc, v = m.nvirt;
  const long nn = static_cast<long>(n) * n, nv = static_cast<long>(n) * v, ov = static_cast<long>(o) * v;
  const bool tdhf = theory == 1;
  const int nb = tdhf ? 2 * kc : kc;
  auto mark = [&](int p) {
    if (ev) SEQX_HIP(hipEventRecord((*ev)[p], st));
  };
  mark(0);
  SigmaEpilogue ep;
  ep.eps = m.eps.p;
  ep.nocc = o;
  ep.V = Vc;
  ep.strideV = ov;
  ep.kv = kc;
  // Outputs interleaved by vector ((A+B)V_I and (A-B)V_I half a row stride
  // apart, as the Davidson basis keeps them): F+ and F- are built
  // interleaved too, so the last product is one launch over all 2 kc
  // matrices (twice the workgroups of a launch per half).
  const bool merged = tdhf && os % 2 == 0 && (io ? io->out2 == io->out1 + os / 2 : out2c == out1c + os / 2);
  const long sF = merged ? 2 * nn : nn;
  const long f2off = merged ? nn : kc * nn;
  if (merged) ep.vdiv = 2;
  if (precision == kPrecFP64) {
    // T1_I (n x v) = C[:, :o] V_I
    dgemm(st, false, false, n, v, o, 1.0, m.C.p, n, 0, Vc, v, ov, 0.0, b.T1, v, nv, kc);
    mark(1);
    // R_I (n x n) = T1_I C[:, o:]^T: the T1_I are stacked rows, so one GEMM with M = kc n
    dgemm(st, false, true, kc * n, n, v, 1.0, b.T1, v, 0, m.C.p + o, n, 0, 0.0, b.R, n, 0, 1);
    mark(2);
    if (tdhf)
      build_G(m, kc, b.R, nn, b.F, b.F + f2off, sF, kTwo, 4.0, -2.0, -2.0, b.gr, b.gJ, b.gws, st);
    else
      build_G(m, kc, b.R, nn, b.F, static_cast<double*>(nullptr), nn, kSum, 2.0, -1.0, -1.0, b.gr, b.gJ, b.gws, st);
    mark(3);
    // Z_b (n x v) = F_b (n x n) * C[:, o:], all nb at once (M = nb n)
    dgemm(st, false, false, nb * n, v, n, 1.0, b.F, n, 0, m.C.p + o, n, 0, 0.0, b.Z, v, 0, 1);
    mark(4);
    // out_b (o x v) = C[:, :o]^T * Z_b + de o V_b
    if (merged) {
      dgemm(st, true, false, o, v, n, 1.0, m.C.p, n, 0, b.Z, v, nv, 0.0, out1c, v, os / 2, nb, &ep);
    } else {
      dgemm(st, true, false, o, v, n, 1.0, m.C.p, n, 0, b.Z, v, nv, 0.0, out1c, v, os, kc, &ep);
      if (tdhf) dgemm(st, true, false, o, v, n, 1.0, m.C.p, n, 0, b.Z + kc * nv, v, nv, 0.0, out2c, v, os, kc, &ep);
    }
  } else if (b.Vp) {
    // bfloat16 planes: every operand with its summation index along the rows,
    // so V enters transposed and Z is formed transposed
    const int np = plane_count(m, precision);
    const long rn = plane_row(n, np), rv = plane_row(v, np), ro = plane_row(o, np);
    if (io) {
      ep.V = nullptr;
      ep.Vf = io->V;
      split_transposed<float>(st, np, kc, o, v, io->V, v, ov, b.Vp);
    } else {
      split_transposed<double>(st, np, kc, o, v, Vc, v, ov, b.Vp);
    }
    // T1_I (n x v) = C_o V_I
    plane_gemm_planes(st, {np, kc, v, n, o, b.Vp, m.Cop.p, v * ro, 0}, b.T1p, n * rv);
    mark(1);
    // R_I (n x n) = T1_I C_v^T over the stacked rows of T1
    plane_gemm_f32(st, {np, 1, n, kc * n, v, m.Cvp.p, b.T1p, 0, 0}, b.Rs, n);
    mark(2);
    const long mat = n * rn, sP = merged ? 2 * mat : mat;
    plane_t* F2 = b.Fp + (merged ? mat : kc * mat);
    if (tdhf)
      build_G_planes(m, kc, b.Rs, nn, np, b.Fp, F2, sP, kTwo, 4.0, -2.0, -2.0, b.gr, b.gJ, b.gws, st);
    else
      build_G_planes(m, kc, b.Rs, nn, np, b.Fp, b.Fp, sP, kSum, 2.0, -1.0, -1.0, b.gr, b.gJ, b.gws, st);
    mark(3);
    // Z_b^T (v x n) = C_v^T F_b^T
    const long zt = v * rn;
    plane_gemm_planes(st, {np, nb, n, v, n, b.Fp, m.CvTp.p, mat, 0}, b.Zp, zt);
    mark(4);
    // out_b (o x v) = C_o^T Z_b + de o V_b
    auto back = [&](int nz, const plane_t* Z, auto* out, long stride) {
      plane_gemm_sigma(st, {np, nz, v, o, n, Z, m.CoTp.p, zt, 0}, out, v, stride, ep);
    };
    auto finish = [&](auto* o1, auto* o2) {
      if (merged) {
        back(nb, b.Zp, o1, os / 2);
      } else {
        back(kc, b.Zp, o1, os);
        if (tdhf) back(kc, b.Zp + kc * zt, o2, os);
      }
    };
    if (io) finish(io->out1, io->out2);
    else finish(out1c, out2c);
  } else {
    // FP32 storage, products on the FP32 matrix cores
    const float* C32 = m.C32.p;
    to_float(st, kc * ov, Vc, b.V32);
    sgemm(st, false, false, n, v, o, 1.0, C32, n, 0, b.V32, v, ov, 0.0, b.T1s, v, nv, kc);
    mark(1);
    sgemm(st, false, true, kc * n, n, v, 1.0, b.T1s, v, 0, C32 + o, n, 0, 0.0, b.Rs, n, 0, 1);
    mark(2);
    if (tdhf)
      build_G(m, kc, b.Rs, nn, b.Fs, b.Fs + f2off, sF, kTwo, 4.0, -2.0, -2.0, b.gr, b.gJ, b.gws, st);
    else
      build_G(m, kc, b.Rs, nn, b.Fs, static_cast<float*>(nullptr), nn, kSum, 2.0, -1.0, -1.0, b.gr, b.gJ, b.gws, st);
    mark(3);
    sgemm(st, false, false, nb * n, v, n, 1.0, b.Fs, n, 0, C32 + o, n, 0, 0.0, b.Zs, v, 0, 1);
    mark(4);
    if (merged) {
      sgemm_out64(st, true, false, o, v, n, 1.0, C32, n, 0, b.Zs, v, nv, 0.0, out1c, v, os / 2, nb, &ep);
    } else {
      sgemm_out64(st, true, false, o, v, n, 1.0, C32, n, 0, b.Zs, v, nv, 0.0, out1c, v, os, kc, &ep);
      if (tdhf) sgemm_out64(st, true, false, o, v, n, 1.0, C32, n, 0, b.Zs + kc * nv, v, nv, 0.0, out2c, v, os, kc, &ep);
    }
  }
  mark(5);
}

void check_sigma_args(const DeviceMolecule& m, int precision) {
  if (precision != kPrecFP64 && precision != kPrecFP32 && precision != kPrecBF16x3)
    throw Error(kEArg, "unsupported transform precision");
  if (precision != kPrecFP64 && m.C32.n < static_cast<size_t>(m.nao) * m.nao)
    throw Error(kEState, "FP32 MO coefficients missing");
}

// Pieces of one chunk's intermediates laid out in a single workspace, each
// starting on a 256-byte boundary; returns the bytes used.  base == nullptr
// only measures.  planes: the plane set instead of the FP32 set; Z then takes
// the place of R, which the contraction has consumed.
size_t carve_chunk(const DeviceMolecule& m, int theory, int kc, int precision, bool planes, unsigned char* base,
                   ChunkBufs* b) {
  const size_t n = m.nao, v = m.nvirt, ov = static_cast<size_t>(m.nocc) * m.nvirt;
  const size_t nn = n * n, nv = n * v, nb = theory == 1 ? 2 * static_cast<size_t>(kc) : kc;
  size_t off = 0;
  auto take = [&](size_t bytes) -> unsigned char* {
    unsigned char* p = base ? base + off : nullptr;
    off += (bytes + 255) / 256 * 256;
    return p;
  };
  ChunkBufs c;
  if (precision == kPrecFP64) {
    c.T1 = reinterpret_cast<double*>(take(kc * nv * sizeof(double)));
    c.R = reinterpret_cast<double*>(take(kc * nn * sizeof(double)));
    c.F = reinterpret_cast<double*>(take(nb * nn * sizeof(double)));
    c.Z = reinterpret_cast<double*>(take(nb * nv * sizeof(double)));
  } else if (planes) {
    const int np = plane_count(m, precision);
    const size_t rn = plane_row(m.nao, np), rv = plane_row(m.nvirt, np), ro = plane_row(m.nocc, np);
    c.Vp = reinterpret_cast<plane_t*>(take(kc * v * ro * sizeof(plane_t)));
    c.T1p = reinterpret_cast<plane_t*>(take(kc * n * rv * sizeof(plane_t)));
    unsigned char* rz = take(std::max(kc * nn * sizeof(float), nb * v * rn * sizeof(plane_t)));
    c.Rs = reinterpret_cast<float*>(rz);
    c.Zp = reinterpret_cast<plane_t*>(rz);
    c.Fp = reinterpret_cast<plane_t*>(take(nb * n * rn * sizeof(plane_t)));
  } else {
    c.V32 = reinterpret_cast<float*>(take(kc * ov * sizeof(float)));
    c.T1s = reinterpret_cast<float*>(take(kc * nv * sizeof(float)));
    c.Rs = reinterpret_cast<float*>(take(kc * nn * sizeof(float)));
    c.Fs = reinterpret_cast<float*>(take(nb * nn * sizeof(float)));
    c.Zs = reinterpret_cast<float*>(take(nb * nv * sizeof(float)));
  }
  const size_t kp = static_cast<size_t>(kc) * m.np;
  c.gr = reinterpret_cast<double*>(take(kp * sizeof(double)));
  c.gJ = reinterpret_cast<double*>(take(kp * sizeof(double)));
  c.gws = reinterpret_cast<double*>(take((g_work_doubles(kc, m.np) - 2 * kp) * sizeof(double)));
  if (b) *b = c;
  return off;
}

// Algorithmic work of one chunk (flops, bytes, launches per phase).  planes: the
// operands C, V, T1, F and Z are rows of that many bfloat16 planes (0: matrices);
// io32: FP32 vectors in and out.
void chunk_work(const DeviceMolecule& m, int theory, int kc, int precision, int planes, bool io32, bool merged,
                std::array<double, kNumPhases>& fl, std::array<double, kNumPhases>& by,
                std::array<long, kNumPhases>& la) {
  const int n = m.nao, o = m.nocc, v = m.nvirt;
  const double nn = static_cast<double>(n) * n, ov = static_cast<double>(o) * v;
  const bool tdhf = theory == 1, low = precision != kPrecFP64;
  const double k = kc, nb = tdhf ? 2.0 * kc : kc;
  const double d = low ? 4.0 : 8.0;  // bytes of an element of a matrix, and of R in any form
  // bytes of an operand of `rows` rows of `len` elements
  auto operand = [&](double rows, int len) { return rows * (planes ? 2.0 * plane_row(len, planes) : d * len); };
  const double T1 = k * operand(n, v), F = nb * operand(n, n), Z = nb * operand(v, n);
  // orbital coefficients always have three planes
  auto orbitals = [&](double rows, int len) { return rows * (planes ? 2.0 * plane_row(len, 3) : d * len); };
  fl = {};
  by = {};
  la = {};
  fl[kPhaseFwd1] = 2.0 * n * ov * k;
  by[kPhaseFwd1] = orbitals(n, o) + k * operand(v, o) + T1;
  fl[kPhaseFwd2] = 2.0 * nn * v * k;
  by[kPhaseFwd2] = orbitals(n, v) + T1 + d * k * nn;
  // contraction: read R, write every F, read the packed ERIs (FP64) once
  by[kPhaseG] = d * k * nn + F + 8.0 * static_cast<double>(m.np) * m.np;
  fl[kPhaseBwd1] = 2.0 * nn * v * nb;
  by[kPhaseBwd1] = orbitals(v, n) + F + Z;
  fl[kPhaseBwd2] = 2.0 * n * ov * nb;
  by[kPhaseBwd2] = orbitals(o, n) + Z + (io32 ? 4.0 : 8.0) * 2.0 * ov * nb;
  la[kPhaseFwd1] = low ? 2 : 1;  // the vectors are split or rounded first
  la[kPhaseFwd2] = 1;
  la[kPhaseG] = 1;
  la[kPhaseBwd1] = 1;
  la[kPhaseBwd2] = tdhf && !merged ? 2 : 1;
}

}  // namespace

namespace {

// FP64 vectors and products (V, out1, out2), or FP32 ones (Vf, out1f, out2f)
void sigma_build_any(const DeviceMolecule& m, int theory, int k, const double* V, double* out1, double* out2,
                     const float* Vf, float* out1f, float* out2f, SigmaWork& w, hipStream_t st, int chunk,
                     long out_stride, int precision) {
  const long ov = static_cast<long>(m.nocc) * m.nvirt;
  const long os = out_stride > 0 ? out_stride : ov;
  const bool tdhf = theory == 1;
  const bool f32io = Vf != nullptr;
  check_sigma_args(m, precision);
  bool has = has_planes(m, precision);
  if (f32io && !has) throw Error(kEArg, "FP32 vectors need plane transforms");
  for (int c0 = 0, kc = 0; c0 < k; c0 += kc) {
    kc = std::min(chunk, k - c0);
    // Where memory is short, fewer vectors at a time, down to one, and then the
    // FP32 matrices (two thirds of the planes): what 32 vectors as FP32 matrices
    // need is always enough.  (Solves over FP32 vectors stop at one: their FP64
    // phase needs more than that vector's planes.)
    bool planes;
    for (;;) {
      planes = has && (f32io || !prefers_matrices(m, theory, kc));
      try {
        w.buf.ensure(carve_chunk(m, theory, kc, precision, planes, nullptr, nullptr));
        break;
      } catch (const Error& e) {
        if (e.status != kENoMem || (kc == 1 && (!planes || f32io))) throw;
        (void)hipGetLastError();  // a failed hipMalloc would be reported by the next launch check
        if (kc > 1) chunk = kc = (kc + 1) / 2;
        else has = false;
      }
    }
    ChunkBufs b;
    carve_chunk(m, theory, kc, precision, planes, w.buf.p, &b);
    std::array<hipEvent_t, kNumPhases + 1> ev;
    for (auto& e : ev) SEQX_HIP(hipEventCreate(&e));
    bool merged;
    if (f32io) {
      F32Io io;
      io.V = Vf + c0 * ov;
      io.out1 = out1f + c0 * os;
      io.out2 = out2f ? out2f + c0 * os : nullptr;
      sigma_chunk(m, theory, kc, nullptr, nullptr, nullptr, os, precision, b, st, &ev, &io);
      merged = tdhf && os % 2 == 0 && io.out2 == io.out1 + os / 2;
    } else {
      double* o1 = out1 + c0 * os;
      double* o2 = out2 ? out2 + c0 * os : nullptr;
      sigma_chunk(m, theory, kc, V + c0 * ov, o1, o2, os, precision, b, st, &ev);
      merged = tdhf && os % 2 == 0 && o2 == o1 + os / 2;
    }
    std::array<double, kNumPhases> fl, by;
    std::array<long, kNumPhases> la;
    chunk_work(m, theory, kc, precision, planes ? plane_count(m, precision) : 0, f32io, merged, fl, by, la);
    w.timer.pending.push_back(ev);
    w.timer.pending_flops.push_back(fl);
    w.timer.pending_bytes.push_back(by);
    w.timer.pending_launches.push_back(la);
  }
}

}  // namespace

void sigma_build(const DeviceMolecule& m, int theory, int k, const double* V, double* out1, double* out2,
                 SigmaWork& w, hipStream_t st, int chunk, long out_stride, int precision) {
  sigma_build_any(m, theory, k, V, out1, out2, nullptr, nullptr, nullptr, w, st, chunk, out_stride, precision);
}

void sigma_build_f32(const DeviceMolecule& m, int theory, int k, const float* V, float* out1, float* out2,
                     SigmaWork& w, hipStream_t st, int chunk, long out_stride, int precision) {
  sigma_build_any(m, theory, k, nullptr, nullptr, nullptr, V, out1, out2, w, st, chunk, out_stride, precision);
}

// ---- no-allocation variant --------------------------------------------------
// One fixed workspace per GPU: a file-scope device array.  Its name is only a
// host-side stand-in for the symbol; the device address of each GPU's copy
// comes from hipGetSymbolAddress (sigma_scratch_setup) and only that address
// is handed to kernels.
static __device__ __align__(256) unsigned char scratch[kSigmaScratchBytes];

namespace {
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxScratchDevices] = {};
}  // namespace

void sigma_scratch_setup(int device) {
  if (device < 0 || device >= kMaxScratchDevices) throw Error(kEDevice, "device index beyond the scratch table");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !p)
    throw Error(kEDevice, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
  g_scratch_ptr[device] = p;
}

namespace {
// vectors per pass that fit the workspace (0: not even one)
int scratch_chunk(const DeviceMolecule& m, int theory, int precision, bool planes) {
  int kc = 32;
  while (kc > 0 && carve_chunk(m, theory, kc, precision, planes, nullptr, nullptr) > kSigmaScratchBytes) --kc;
  return kc;
}
}  // namespace

void sigma_build_noalloc(const DeviceMolecule& m, int theory, int k, const double* V, double* out1, double* out2,
                         hipStream_t st, int precision) {
  check_sigma_args(m, precision);
  int device = 0;
  SEQX_HIP(hipGetDevice(&device));
  void* base = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (device >= 0 && device < kMaxScratchDevices) base = g_scratch_ptr[device];
  }
  if (!base) {
    sigma_scratch_setup(device);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    base = g_scratch_ptr[device];
  }
  // the plane set where one vector of it fits; the FP32 set is smaller and
  // reaches up to about 2800 AOs
  bool planes = has_planes(m, precision);
  int chunk = scratch_chunk(m, theory, precision, planes);
  if (chunk < 1 && planes) {
    planes = false;
    chunk = scratch_chunk(m, theory, precision, false);
  }
  if (chunk < 1)
    throw Error(kEBufSize, "one trial vector needs " +
                               std::to_string(carve_chunk(m, theory, 1, precision, planes, nullptr, nullptr)) +
                               " bytes of intermediates; the fixed workspace holds " +
                               std::to_string(kSigmaScratchBytes));
  const long ov = static_cast<long>(m.nocc) * m.nvirt;
  for (int c0 = 0; c0 < k; c0 += chunk) {
    const int kc = std::min(chunk, k - c0);
    ChunkBufs b;
    carve_chunk(m, theory, kc, precision, planes && !prefers_matrices(m, theory, kc), static_cast<unsigned char*>(base),
                &b);
    sigma_chunk(m, theory, kc, V + c0 * ov, out1 + c0 * ov, out2 ? out2 + c0 * ov : nullptr, ov, precision, b, st,
                nullptr);
  }
}

}  // namespace seqx
