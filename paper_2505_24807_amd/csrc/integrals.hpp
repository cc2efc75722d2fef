// NDDO integral tables and core Hamiltonian on the device.
#pragma once

#include "molecule.hpp"

namespace seqx {

// Fill m.W (packed ERIs, every block written) and m.H (core Hamiltonian,
// every element written) from the molecule's geometry and element table.
void build_integrals(const DeviceMolecule& m, hipStream_t st);
// The same tables from ntab other device element tables (kNumSlots entries
// each), into W [ntab][np][np] and H [ntab][nao][nao].
void build_integrals(const DeviceMolecule& m, const Elem* elems, double* W, double* H, hipStream_t st, int ntab);

}  // namespace seqx
