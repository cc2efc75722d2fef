"""Projected problems of exactly the sizes where the subspace eigensolver changes
its kernels: the first Ritz values of a guess of n vectors against NumPy.

The guess also makes the n x n Gram matrix of which all pairs are wanted.
"""
import numpy as np
import pytest

from paper_2505_24807_amd import seqx
from synthetic import molecules, params

pytestmark = pytest.mark.gpu
PR = params.load()


@pytest.fixture(scope="module")
def prepared():
    """C20H22 (2601 pairs) and its matrices, from products of unit vectors."""
    ctx = seqx.Context(0)
    ctx.set_params(*seqx.params_table(PR))
    mol = molecules.add_noise(molecules.polyene(20), 0.02, np.random.default_rng(20))
    job = ctx.prepare([mol.natoms], mol.Z, mol.xyz)
    n, o, v = job.dims()
    unit = np.eye(o * v).reshape(o * v, o, v)
    A = job.sigma(unit, theory=seqx.CIS)[0].reshape(o * v, o * v)
    P, M = (x.reshape(o * v, o * v) for x in job.sigma(unit, theory=seqx.TDHF))
    yield job, o, v, {seqx.CIS: (A,), seqx.TDHF: (P, M)}
    job.free()
    ctx.close()


# edges of Jacobi (12), of one, two, three, four, six and eight blocks of 64 columns, of the reduction in one workgroup
# (128) and of the whole solver (512); 48 and 256 bound the Jacobi and Cholesky kernels
@pytest.mark.parametrize("n", [12, 13, 48, 49, 64, 65, 128, 129, 192, 193, 256, 257, 384, 385, 512, 513])
@pytest.mark.parametrize("theory", [seqx.CIS, seqx.TDHF])
def test_first_ritz_values(prepared, n, theory):
    """FP64 projections and eigensolves of matrices of order one: 1e-9 eV leaves four orders above their rounding."""
    job, o, v, mats = prepared
    print(f"[gpu] subspace of {n} rows theory={theory}", flush=True)
    guess = np.random.default_rng(n).normal(size=(n, o * v))
    Q = np.linalg.qr(guess.T)[0]
    proj = [Q.T @ A @ Q for A in mats[theory]]
    proj = [(x + x.T) / 2 for x in proj]
    k = 4
    if theory == seqx.CIS:
        ref = np.linalg.eigvalsh(proj[0])[:k]
    else:
        L = np.linalg.cholesky(proj[1])
        ref = np.sqrt(np.linalg.eigvalsh(L.T @ proj[0] @ L)[:k])
    job.solve(theory=theory, nroots=k, tol=1e-2, max_iter=300, guess=seqx.GUESS_USER,
              user_guess=guess.reshape(n, o, v), max_subspace=n + 16)
    assert job.stats().max_subspace_used >= n
    assert np.abs(job.history()[1][0] - ref * seqx.HARTREE_EV).max() <= 1e-9
