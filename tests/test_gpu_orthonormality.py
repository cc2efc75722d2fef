"""The Davidson basis stays orthonormal: solves of clusters whose corrections lie
largely in the basis and nearly repeat each other (a dense band of close roots
over more than a hundred iterations).

A basis that loses orthogonality from iteration to iteration ends with roots at
zero, vectors of norm zero, or a projected matrix that is not positive definite.
"""
import numpy as np
import pytest

from paper_2505_24807_amd import seqx
from synthetic import molecules, params

pytestmark = pytest.mark.gpu
PR = params.load()


@pytest.fixture(scope="module")
def ctx():
    c = seqx.Context(0)
    c.set_params(*seqx.params_table(PR))
    yield c
    c.close()


def _norms(r):
    X, Y = r.X.reshape(len(r.X), -1), r.Y.reshape(len(r.Y), -1)
    return np.abs(X @ X.T - Y @ Y.T - np.eye(len(X))).max()


# basis rows of FP32 (pairs a multiple of four, at least 4096) in the low-precision phase; the reference keeps FP64
@pytest.mark.parametrize("n_water, seed, theory", [(40, 40001, seqx.CIS), (40, 40002, seqx.CIS), (80, 80000, seqx.CIS),
                                                   (40, 40002, seqx.TDHF), (80, 80000, seqx.TDHF)])
def test_low_precision_solve_of_a_dense_band(ctx, n_water, seed, theory):
    """Mixed solves find the roots of the FP64 solve.  Residuals below 1e-6 hartree bound an eigenvalue's error by as
    much (CIS), in TDHF by a few times it: bar 1e-4 eV, 1e-12 for the norms."""
    mol = molecules.water_cluster(n_water, seed)
    print(f"[gpu] dense band {mol.name} theory={theory}", flush=True)
    job = ctx.prepare([mol.natoms], mol.Z, mol.xyz)
    job.solve(theory=theory, nroots=8, tol=1e-8, max_iter=600)
    ref = job.results()
    assert _norms(ref) <= 1e-12
    for precision in (seqx.FP32, seqx.BF16X3):
        job.solve(theory=theory, nroots=8, tol=1e-6, max_iter=600, precision=precision)
        got = job.results()
        assert np.abs(got.omega_eV - ref.omega_eV).max() <= 1e-4
        assert _norms(got) <= 1e-12
    job.free()


@pytest.mark.parametrize("n_water, seed", [(11, 11000), (16, 16004), (20, 20004)])
def test_fp64_vectors_are_orthonormal(ctx, n_water, seed):
    """FP64 solves over FP64 rows: norms and overlaps of the vectors to 1e-12 (sums of up to 3200 terms round to 1e-14)."""
    mol = molecules.water_cluster(n_water, seed)
    print(f"[gpu] orthonormal vectors {mol.name}", flush=True)
    job = ctx.prepare([mol.natoms], mol.Z, mol.xyz)
    job.solve(theory=seqx.CIS, nroots=7, tol=1e-8, max_iter=600)
    assert _norms(job.results()) <= 1e-12
    job.free()


def test_guess_of_nearly_dependent_vectors(ctx):
    """A guess whose second half repeats the first to 1e-5: its Gram matrix has eigenvalues near 1e-10, and the basis
    must still be orthonormal for the first Ritz values to be those of the span (FP64 QR of the guess)."""
    mol = molecules.water_cluster(11, 11)
    print(f"[gpu] nearly dependent guess {mol.name}", flush=True)
    job = ctx.prepare([mol.natoms], mol.Z, mol.xyz)
    n, o, v = job.dims()
    rng = np.random.default_rng(7)
    half = rng.normal(size=(8, o, v))
    guess = np.concatenate([half, half + 1e-5 * rng.normal(size=half.shape)])
    Q = np.linalg.qr(guess.reshape(16, -1).T)[0].T.reshape(16, o, v)
    AQ, _ = job.sigma(Q, theory=seqx.CIS)
    M = Q.reshape(16, -1) @ AQ.reshape(16, -1).T
    job.solve(theory=seqx.CIS, nroots=4, tol=1e-6, max_iter=300, guess=seqx.GUESS_USER, user_guess=guess)
    first = job.history()[1][0]
    # the span itself is known to 2^-52 / 1e-5 of a vector
    assert np.abs(first - np.linalg.eigvalsh((M + M.T) / 2)[:4] * seqx.HARTREE_EV).max() <= 1e-8
    job.free()


@pytest.mark.parametrize("theory, k", [(seqx.TDHF, 8), (seqx.TDHF, 5), (seqx.CIS, 8)])
def test_whole_space(ctx, theory, k):
    """Water has 8 pairs: more corrections (2 k) than the space has dimensions.  No tolerance of 1e-300 is reached and
    no direction is left (E_DAV_NOCONV); the next solve finds all roots."""
    mol = molecules.water_cluster(1, 1)
    print(f"[gpu] whole space theory={theory} k={k}", flush=True)
    job = ctx.prepare([mol.natoms], mol.Z, mol.xyz)
    n, o, v = job.dims()
    assert o * v == 8
    with pytest.raises(seqx.SeqxError) as ei:
        job.solve(theory=theory, nroots=k, tol=1e-300, max_iter=5)
    assert ei.value.status == 8
    job.solve(theory=theory, nroots=k, tol=1e-8)
    P, M = job.sigma(np.eye(8).reshape(8, o, v), theory=theory)
    if theory == seqx.CIS:
        ref = np.linalg.eigvalsh(P.reshape(8, 8))
    else:
        L = np.linalg.cholesky(M.reshape(8, 8))
        ref = np.sqrt(np.linalg.eigvalsh(L.T @ P.reshape(8, 8) @ L))
    assert np.abs(job.results().omega_eV - ref[:k] * seqx.HARTREE_EV).max() <= 1e-10
    job.free()
