"""A Householder reduction whose wavefronts on different compute units wait for
each other gives up after a bounded number of polls (other work may hold the
GPU); the solve then takes the dense library and returns the same roots.

The limit is set to nothing from the host (SEQX_EIG_POLL_LIMIT), so that the
wait ends at its first poll.
"""
import numpy as np
import pytest

from oracle import excited, integrals, model, scf
from paper_2505_24807_amd import seqx
from synthetic import molecules, params

pytestmark = pytest.mark.gpu
PR = params.load()


# Gram matrices of up to 140 new directions and subspaces of more than 128 rows, both above one workgroup's reduction
@pytest.mark.parametrize("theory, k", [(seqx.CIS, 140), (seqx.TDHF, 70)])
def test_solve_without_the_reduction(monkeypatch, theory, k):
    """Residuals below 1e-6 hartree bound the error of a CIS root by as much, of a TDHF root by a few times it: 1e-4 eV."""
    monkeypatch.setenv("SEQX_EIG_POLL_LIMIT", "0")
    mol = molecules.add_noise(molecules.polyene(20), 0.02, np.random.default_rng(20))
    print(f"[gpu] reduction gives up {mol.name} theory={theory} k={k}", flush=True)
    ctx = seqx.Context(0)
    ctx.set_params(*seqx.params_table(PR))
    job = ctx.prepare([mol.natoms], mol.Z, mol.xyz)
    n, o, v = job.dims()
    job.solve(theory=theory, nroots=k, tol=1e-6, max_iter=100)
    got = job.results()
    sy = model.make_system(mol.Z, mol.xyz, PR)
    ints = integrals.build(sy)
    res = scf.run(sy, ints)
    A, B = excited.build_AB(ints, res.eps, res.C, o)
    ref = excited.cis_dense(A, k, o, v) if theory == seqx.CIS else excited.tdhf_dense(A, B, k, o, v)
    assert np.abs(got.omega_eV - ref.omega * model.HARTREE_EV).max() <= 1e-4
    job.free()
    ctx.close()


@pytest.mark.parametrize("bits", [0x7FF8000000000000, 0xFFF8000000000000, 0xFFFFFFFFFFFFFFFF])
def test_guess_with_a_nan(bits):
    """A guess of more than 128 vectors with a NaN of any kind is refused, and at once: the reduction does not take the
    NaN for a value still to come (a wait of seconds)."""
    import time

    mol = molecules.add_noise(molecules.polyene(20), 0.02, np.random.default_rng(20))
    print(f"[gpu] guess with a NaN {bits:x}", flush=True)
    ctx = seqx.Context(0)
    ctx.set_params(*seqx.params_table(PR))
    job = ctx.prepare([mol.natoms], mol.Z, mol.xyz)
    n, o, v = job.dims()
    guess = np.random.default_rng(1).normal(size=(140, o, v))
    t0 = time.perf_counter()
    job.solve(theory=seqx.CIS, nroots=4, tol=1e-3, max_iter=300, guess=seqx.GUESS_USER, user_guess=guess,
              max_subspace=300)
    usual = time.perf_counter() - t0
    guess[5] = np.full((o, v), bits, dtype=np.uint64).view(np.float64)
    t0 = time.perf_counter()
    with pytest.raises(seqx.SeqxError) as ei:
        job.solve(theory=seqx.CIS, nroots=4, tol=1e-3, max_iter=300, guess=seqx.GUESS_USER, user_guess=guess,
                  max_subspace=300)
    assert ei.value.status == 1  # E_ARG: no direction left
    assert time.perf_counter() - t0 < usual + 0.3
    job.free()
    ctx.close()
