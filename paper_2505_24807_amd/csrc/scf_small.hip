// Ground states of small molecules (n <= kScfSmallMax AOs), one workgroup per
// molecule and one launch for all of them: the whole SCF iteration of scf.hip
// (NDDO Fock matrix, DIIS, SP2 purification) runs inside the workgroup.
//
// A molecule of 12-136 AOs takes about 17 cycles of 20 purification steps;
// launched one by one these are some 3000 launches a molecule, and the launches
// set the time however many molecules run side by side.  Here the matrix that
// is purified stays in LDS (n <= 136: 153 KB), a step is one symmetric product
// on the FP64 matrix cores with the update in its epilogue, and the other
// matrices stay in L2.  128 molecules of 12-136 AOs (their ground
// states with set-up, integrals and final eigensolves): 355 -> 130 ms; this
// kernel takes 3.4 ms for an average molecule alone.
#include <algorithm>
#include <cmath>

#include "diis.hpp"
#include "fock_blocks.hpp"
#include "scf.hpp"
#include "wave.hpp"

namespace seqx {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kST = 512;        // threads per molecule
constexpr int kSW = kST / 64;
// LDS row stride of the purified matrix: an odd multiple of 16 doubles, so that
// the four rows of one operand read start in alternate halves of the banks
constexpr int kSLd = 144;
constexpr int kSTiles = 6;      // 16 x 16 tiles of the upper triangle per wavefront: 45 / 8

struct ScfDesc {
  int n, o, np, natoms, npairs[3];
  const int *slot, *ao_off, *pi_off, *pi_mu, *pi_nu, *atom_of_ao;
  const int2* pairs[3];
  const Elem* elems;
  const double *W, *H;
  double *P, *F;         // outputs: density, converged Fock matrix
  double *FP, *Fh, *Eh;  // work: n x n, nd histories of n x n each
  double* out;           // max |FP - PF|, cycles, status (0 converged, 1 not, 2 NaN)
};

struct ScfLds {
  double X[kScfSmallMax][kSLd];  // purification; packed densities and Coulomb values in between
  double red[2 * kSW];
  double B[kDiisMax][kDiisMax + 1], c[kDiisMax];
  double lo[kSW], hi[kSW];
  DiisLds diis;
};

// sums of two values over the workgroup in a fixed order (every thread gets them)
__device__ void wg_sum2(double& x, double& y, double* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  x = wave_sum64(x);
  y = wave_sum64(y);
  __syncthreads();  // red may still be read from the previous call
  if (lane == 0) {
    red[2 * wave] = x;
    red[2 * wave + 1] = y;
  }
  __syncthreads();
  x = 0.0;
  y = 0.0;
  for (int w = 0; w < kSW; ++w) {
    x += red[2 * w];
    y += red[2 * w + 1];
  }
}

__device__ double wave_max64(double x) {
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) x = fmax(x, __shfl_xor(x, m));
  return x;
}

// F = H + J(P) - K(P) / 2; P symmetric
__device__ void small_fock(const ScfDesc& m, const double* P, ScfLds& L) {
  const int n = m.n, np = m.np, tid = threadIdx.x;
  double* rs = &L.X[0][0];
  double* js = rs + np;
  for (int q = tid; q < np; q += kST) {
    const int mu = m.pi_mu[q], nu = m.pi_nu[q];
    const double x = P[mu * n + nu];
    rs[q] = mu == nu ? x : x + P[nu * n + mu];
  }
  __syncthreads();
  for (int q = tid; q < np; q += kST) {  // W symmetric: column q, coalesced over the threads
    const double* w = m.W + q;
    double s[4] = {0, 0, 0, 0};
    int r = 0;
    for (; r + 4 <= np; r += 4)
#pragma unroll
      for (int u = 0; u < 4; ++u) s[u] += w[static_cast<long>(r + u) * np] * rs[r + u];
    for (; r < np; ++r) s[0] += w[static_cast<long>(r) * np] * rs[r];
    js[q] = (s[0] + s[1]) + (s[2] + s[3]);
  }
  __syncthreads();
  const MatOut<double> F{m.F, 0, n};
  for (int A = tid; A < m.natoms; A += kST)
    diag_block<kSymm, double>(m.elems[m.slot[A]], m.ao_off[A], m.pi_off[A], js, 1, P, n, F, F, 1.0, -0.5, 0.0);
  for (int p = tid; p < m.npairs[0]; p += kST)
    exchange_pair<4, 4, kSymm, double, double>(m.pairs[0][p].x, m.pairs[0][p].y, m.ao_off, m.pi_off, m.W, np, P, n,
                                               m.F, nullptr, -0.5, 0.0);
  for (int p = tid; p < m.npairs[1]; p += kST)
    exchange_pair<4, 1, kSymm, double, double>(m.pairs[1][p].x, m.pairs[1][p].y, m.ao_off, m.pi_off, m.W, np, P, n,
                                               m.F, nullptr, -0.5, 0.0);
  for (int p = tid; p < m.npairs[2]; p += kST)
    exchange_pair<1, 1, kSymm, double, double>(m.pairs[2][p].x, m.pairs[2][p].y, m.ao_off, m.pi_off, m.W, np, P, n,
                                               m.F, nullptr, -0.5, 0.0);
  __syncthreads();
  for (int x = tid; x < n * n; x += kST) m.F[x] += m.H[x];
  __syncthreads();
}

// SP2 purification of Fx into P = 2 X: X <- X^2 or 2 X - X^2, whichever keeps
// tr X closer to the number of occupied orbitals, until X is idempotent.  X is
// symmetric, so tr X^2 is the sum of its squared elements: the branch of a step
// is known before its product, which therefore ends in the new X.
__device__ void small_sp2(const ScfDesc& m, const double* Fx, ScfLds& L) {
  const int n = m.n, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, k4 = lane >> 4;
  const int nt = (n + 15) / 16, ntile = nt * (nt + 1) / 2, kpad = (n + 3) / 4 * 4;
  // Gershgorin bounds: rows over the wavefronts
  double lo = 1e300, hi = -1e300;
  for (int i = wave; i < n; i += kSW) {
    double s = 0.0;
    for (int j = lane; j < n; j += 64) s += j == i ? 0.0 : fabs(Fx[i * n + j]);
    s = wave_sum64(s);
    const double d = Fx[i * n + i];
    lo = fmin(lo, d - s);
    hi = fmax(hi, d + s);
  }
  if (lane == 0) {
    L.lo[wave] = lo;
    L.hi[wave] = hi;
  }
  __syncthreads();
  for (int w = 0; w < kSW; ++w) {
    lo = fmin(lo, L.lo[w]);
    hi = fmax(hi, L.hi[w]);
  }
  // X = (hi I - F) / (hi - lo), zero past n
  double tx = 0.0, tx2 = 0.0;
  const double inv = 1.0 / (hi - lo);
  for (int x = tid; x < kpad * kSLd; x += kST) {
    const int i = x / kSLd, j = x % kSLd;
    double v = 0.0;
    if (i < n && j < n) {
      v = ((i == j ? hi : 0.0) - Fx[i * n + j]) * inv;
      if (i == j) tx += v;
      tx2 += v * v;
    }
    L.X[i][j] = v;
  }
  wg_sum2(tx, tx2, L.red);  // its barriers also publish X
  double e1 = 1e300, e2 = 1e300;
  for (int it = 0; it < 200; ++it) {
    const double e = tx - tx2;  // sum of lambda (1 - lambda) >= 0
    if (!(e > 1e-13 * n) || (e < 1e-6 && e >= e2)) break;
    e2 = e1;
    e1 = e;
    const bool square = fabs(tx2 - m.o) < fabs(2.0 * tx - tx2 - m.o);
    d4 acc[kSTiles];
#pragma unroll
    for (int q = 0; q < kSTiles; ++q) {
      const int t = wave + kSW * q;
      acc[q] = d4{0, 0, 0, 0};
      if (t < ntile) {  // uniform
        int J = 0;      // tile (I, J), I <= J, t = J (J + 1) / 2 + I
        while ((J + 1) * (J + 2) / 2 <= t) ++J;
        const int I = t - J * (J + 1) / 2;
        const double* xa = &L.X[k4][16 * I + r16];
        const double* xb = &L.X[k4][16 * J + r16];
        for (int k = 0; k < kpad; k += 4)
          acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[k * kSLd], xb[k * kSLd], acc[q], 0, 0, 0);
      }
    }
    __syncthreads();
    tx = 0.0;
    tx2 = 0.0;
#pragma unroll
    for (int q = 0; q < kSTiles; ++q) {
      const int t = wave + kSW * q;
      if (t < ntile) {
        int J = 0;
        while ((J + 1) * (J + 2) / 2 <= t) ++J;
        const int I = t - J * (J + 1) / 2;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = 16 * I + k4 + 4 * r, j = 16 * J + r16;
          if (i < n && j < n) {
            const double v = square ? acc[q][r] : 2.0 * L.X[i][j] - acc[q][r];
            if (i == j) tx += v;
            tx2 += I == J ? v * v : 2.0 * v * v;
            L.X[i][j] = v;
            if (I != J) L.X[j][i] = v;
          }
        }
      }
    }
    wg_sum2(tx, tx2, L.red);
  }
  for (int x = tid; x < n * n; x += kST) m.P[x] = 2.0 * L.X[x / n][x % n];
  __syncthreads();
}

// out (n x n) = A B, row-major; operands from L2 in the MFMA lane layout
__device__ void small_product(int n, const double* __restrict__ A, const double* __restrict__ B,
                              double* __restrict__ out) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, k4 = lane >> 4, nt = (n + 31) / 32;
  for (int t = wave; t < nt * nt; t += kSW) {
    const int i0 = (t / nt) * 32, j0 = (t % nt) * 32;
    d4 acc[2][2] = {{d4{0, 0, 0, 0}, d4{0, 0, 0, 0}}, {d4{0, 0, 0, 0}, d4{0, 0, 0, 0}}};
    for (int k0 = 0; k0 < n; k0 += 16) {
      double a[4][2], b[4][2];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = k0 + 4 * q + k4;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int i = i0 + 16 * u + r16, j = j0 + 16 * u + r16;
          a[q][u] = (i < n && k < n) ? A[i * n + k] : 0.0;
          b[q][u] = (j < n && k < n) ? B[k * n + j] : 0.0;
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int w = 0; w < 2; ++w)
            acc[u][w] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q][u], b[q][w], acc[u][w], 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int w = 0; w < 2; ++w)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = i0 + 16 * u + k4 + 4 * r, j = j0 + 16 * w + r16;
          if (i < n && j < n) out[i * n + j] = acc[u][w][r];
        }
  }
  __syncthreads();
}

__global__ void __launch_bounds__(kST) scf_small_kernel(const ScfDesc* __restrict__ mols, double tol, int max_iter,
                                                        int nd) {
  __shared__ ScfLds L;
  const ScfDesc m = mols[blockIdx.x];
  const int n = m.n, nn = n * n, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // diagonal guess: each atom's core charge spread over its AOs
  for (int x = tid; x < nn; x += kST) {
    const int i = x / n;
    double v = 0.0;
    if (i == x % n) {
      const Elem& e = m.elems[m.slot[m.atom_of_ao[i]]];
      v = e.core / e.nao;
    }
    m.P[x] = v;
  }
  __syncthreads();
  small_fock(m, m.P, L);
  small_sp2(m, m.F, L);
  double err = 1e300;
  int it = 1, count = 0, status = 1;
  for (; it <= max_iter; ++it) {
    small_fock(m, m.P, L);
    small_product(n, m.F, m.P, m.FP);
    // commutator F P - P F = X - X^T with X = F P, into its history slot
    const int slot = nd > 1 ? count % nd : 0;
    double* E = m.Eh + static_cast<long>(slot) * nn;
    double mx = 0.0, nans = 0.0, unused = 0.0;
    for (int x = tid; x < nn; x += kST) {
      const int i = x / n, j = x % n;
      const double v = m.FP[x] - m.FP[j * n + i];
      E[x] = v;
      mx = fmax(mx, fabs(v));
      if (!(v == v)) nans = 1.0;
    }
    mx = wave_max64(mx);
    if (lane == 0) L.hi[wave] = mx;
    wg_sum2(nans, unused, L.red);
    err = 0.0;
    for (int w = 0; w < kSW; ++w) err = fmax(err, L.hi[w]);
    __syncthreads();  // L.hi is written again by the purification
    if (nans > 0.0) {
      status = 2;
      break;
    }
    if (err <= tol) {
      status = 0;
      break;
    }
    const double* Fx = m.F;
    if (nd > 1) {
      double* Fs = m.Fh + static_cast<long>(slot) * nn;
      for (int x = tid; x < nn; x += kST) Fs[x] = m.F[x];
      ++count;
      const int mh = min(count, nd);
      // overlaps of the new error matrix with the others, one wavefront each
      for (int s = wave; s < mh; s += kSW) {
        const double* Es = m.Eh + static_cast<long>(s) * nn;
        double d[4] = {0, 0, 0, 0};
        int x = lane;
        for (; x + 192 < nn; x += 256)
#pragma unroll
          for (int u = 0; u < 4; ++u) d[u] += E[x + 64 * u] * Es[x + 64 * u];
        for (; x < nn; x += 64) d[0] += E[x] * Es[x];
        const double v = wave_sum64((d[0] + d[1]) + (d[2] + d[3]));
        if (lane == 0) {
          L.B[slot][s] = v;
          L.B[s][slot] = v;
        }
      }
      __syncthreads();
      if (mh >= 2) {
        diis_solve(mh, &L.B[0][0], kDiisMax + 1, L.c, L.diis);
        for (int x = tid; x < nn; x += kST) {
          double v = 0.0;
          for (int s = 0; s < mh; ++s) v += L.c[s] * m.Fh[static_cast<long>(s) * nn + x];
          m.FP[x] = v;
        }
        __syncthreads();
        Fx = m.FP;
      }
    }
    small_sp2(m, Fx, L);
  }
  if (tid == 0) {
    m.out[0] = err;
    m.out[1] = it;
    m.out[2] = status;
  }
}

}  // namespace

void run_scf_small(const std::vector<DeviceMolecule*>& ms, const ScfOptions& opt, ScfSmallWork& w, hipStream_t st) {
  const int nd = std::max(1, std::min(opt.ndiis, kDiisMax));
  // molecules per launch: one per compute unit, and histories below about 1 GB
  constexpr size_t kPerLaunch = 256;
  constexpr size_t kMaxWork = (size_t(1) << 30) / sizeof(double);
  for (size_t m0 = 0; m0 < ms.size();) {
    size_t m1 = m0, need = 0;
    while (m1 < ms.size() && m1 - m0 < kPerLaunch) {
      const size_t nn = static_cast<size_t>(ms[m1]->nao) * ms[m1]->nao, add = (1 + 2 * static_cast<size_t>(nd)) * nn;
      if (m1 > m0 && need + add > kMaxWork) break;
      need += add;
      ++m1;
    }
    const size_t cnt = m1 - m0;
    w.work.ensure(need);
    w.out.ensure(3 * cnt);
    w.desc.ensure(cnt * sizeof(ScfDesc));
    std::vector<ScfDesc> ds(cnt);
    double* p = w.work.p;
    for (size_t q = 0; q < cnt; ++q) {
      DeviceMolecule& m = *ms[m0 + q];
      if (m.nao > kScfSmallMax || 2 * m.np > kScfSmallMax * kSLd) throw Error(kEArg, "molecule too large for one workgroup");
      const size_t nn = static_cast<size_t>(m.nao) * m.nao;
      m.C.ensure(nn);
      m.P.ensure(nn);
      ScfDesc& d = ds[q];
      d.n = m.nao;
      d.o = m.nocc;
      d.np = m.np;
      d.natoms = m.natoms;
      for (int g = 0; g < 3; ++g) {
        d.npairs[g] = m.npairs[g];
        d.pairs[g] = m.pairs[g].p;
      }
      d.slot = m.slot.p;
      d.ao_off = m.ao_off.p;
      d.pi_off = m.pi_off.p;
      d.pi_mu = m.pi_mu.p;
      d.pi_nu = m.pi_nu.p;
      d.atom_of_ao = m.atom_of_ao.p;
      d.elems = m.elems;
      d.W = m.W.p;
      d.H = m.H.p;
      d.P = m.P.p;
      d.F = m.C.p;  // the orbitals of F replace it afterwards
      d.FP = p;
      d.Fh = p + nn;
      d.Eh = p + (1 + nd) * nn;
      p += (1 + 2 * static_cast<size_t>(nd)) * nn;
      d.out = w.out.p + 3 * q;
    }
    SEQX_HIP(hipMemcpyAsync(w.desc.p, ds.data(), cnt * sizeof(ScfDesc), hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(scf_small_kernel, dim3(cnt), dim3(kST), 0, st, reinterpret_cast<const ScfDesc*>(w.desc.p),
                       opt.tol, opt.max_iter, nd);
    SEQX_LAUNCH_CHECK();
    std::vector<double> out(3 * cnt);
    SEQX_HIP(hipMemcpyAsync(out.data(), w.out.p, out.size() * sizeof(double), hipMemcpyDeviceToHost, st));
    SEQX_HIP(hipStreamSynchronize(st));
    for (size_t q = 0; q < cnt; ++q) {
      DeviceMolecule& m = *ms[m0 + q];
      m.commutator = out[3 * q];
      m.scf_iterations = static_cast<int>(out[3 * q + 1]);
      if (out[3 * q + 2] == 2.0) throw Error(kEScfNoConv, "SCF produced NaN");
      if (out[3 * q + 2] != 0.0)
        throw Error(kEScfNoConv, "SCF did not converge: max|FP-PF| = " + std::to_string(m.commutator));
    }
    m0 = m1;
  }
}

}  // namespace seqx
