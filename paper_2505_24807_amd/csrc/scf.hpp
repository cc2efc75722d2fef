// Closed-shell RHF ground state on the device (Eq. 1 of the paper, S = I).
#pragma once

#include "fock.hpp"
#include "linalg.hpp"
#include "molecule.hpp"

namespace seqx {

struct ScfOptions {
  double tol = 1e-10;
  int max_iter = 300;
  int ndiis = 8;
  bool purify = true;  // density from SP2 purification in the SCF loop (one eigensolve at the end)
};

struct ScfWork {
  DBuf<double> G, F, FP, E, CT, Fhist, Ehist, B, c, scal, red, X2;
  DBuf<float> X32, X2_32;  // FP32 purification steps
};

// Molecules up to this many AOs run their SCF in one workgroup each
// (run_scf_small, then finish_scf); their results do not depend on how many run
// together.
constexpr int kScfSmallMax = 136;
inline bool scf_is_small(const DeviceMolecule& m, const ScfOptions& opt) {
  return opt.purify && m.nao <= kScfSmallMax;
}

struct ScfSmallWork {
  DBuf<double> work, out;
  DBuf<unsigned char> desc;
};

// SCF of every molecule of the list (scf_is_small), one launch for up to 256:
// fills m.P, leaves the converged Fock matrix in m.C; throws Error(kEScfNoConv).
void run_scf_small(const std::vector<DeviceMolecule*>& ms, const ScfOptions& opt, ScfSmallWork& w, hipStream_t st);
// Orbitals of the converged Fock matrix F (n x n, may be m.C itself): fills
// m.C, m.C32, m.eps, m.P and the orbital planes.
void finish_scf(DeviceMolecule& m, const double* F, DenseSolver& ds, ScfWork& w, hipStream_t st);

// Fills m.C (row-major [mu][p]), m.eps, m.P; throws Error(kEScfNoConv) on failure.
void run_scf(DeviceMolecule& m, const ScfOptions& opt, DenseSolver& ds, GWork& gw, ScfWork& w, hipStream_t st);

}  // namespace seqx
