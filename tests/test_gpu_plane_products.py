"""Low-precision products held to the accuracy of their planes: a plane or a
partial product that went missing would show.

The error of the two-electron part, as a norm over the whole product, was worked
out on the CPU for the same chains (C_o V, C_v^T, contraction, C_v, C_o^T) with
FP32 sums: three planes 2.5 to 3.4 times 2^-24; without the lowest plane 88 to
123 times, without the product of the middle planes 59 to 90 times, either in one
of the four transforms alone half as much.  Two planes: 0.42 to 0.61 times 2^-16;
one plane 238 times or more.  Bars: 10 * 2^-24 and 2 * 2^-16.
"""
import numpy as np
import pytest

from oracle import model
from paper_2505_24807_amd import seqx
from synthetic import molecules, params

pytestmark = pytest.mark.gpu
PR = params.load()


# smallest plane transforms (96 AOs, 64 and 32 orbitals), odd numbers (102: 51 and 51), and large ones with an odd
# number of vectors, a full pass of them and one; the split keeps three planes below 96 orbitals and for odd numbers
@pytest.mark.parametrize("mol, k, split_planes",
                         [(molecules.water_cluster(16, 16), 3, 3),
                          (molecules.add_noise(molecules.polyene(20), 0.02, np.random.default_rng(20)), 5, 3),
                          (molecules.water_cluster(67, 67), 7, 2), (molecules.water_cluster(67, 67), 32, 2),
                          (molecules.water_cluster(67, 67), 1, 2)], ids=lambda x: getattr(x, "name", str(x)))
@pytest.mark.parametrize("theory", [seqx.CIS, seqx.TDHF])
def test_plane_products(mol, k, split_planes, theory):
    print(f"[gpu] plane products {mol.name} k={k} theory={theory}", flush=True)
    ctx = seqx.Context(0)
    ctx.set_params(*seqx.params_table(PR))
    job = ctx.prepare([mol.natoms], mol.Z, mol.xyz)
    n, o, v = job.dims()
    eps = job.scf_results()[0] / model.HARTREE_EV
    V = np.random.default_rng(2).normal(size=(k, o, v))
    diag = (eps[None, o:] - eps[:o, None]) * V
    ref = [x for x in job.sigma(V, theory=theory) if x is not None]
    for precision, planes in ((seqx.FP32, 3), (seqx.BF16X3, split_planes)):
        bar = 10 * 2.0 ** -24 if planes == 3 else 2 * 2.0 ** -16
        got = [x for x in job.sigma(V, theory=theory, precision=precision) if x is not None]
        for a, b in zip(got, ref):
            assert np.linalg.norm(a - b) <= bar * np.linalg.norm(b - diag)
    job.free()
    ctx.close()


# the last and first number of vectors on either side of the rule (2 n / 11 vectors, 150 AOs), and a pass of 32 after 8
@pytest.mark.parametrize("mol, k", [(molecules.water_cluster(16, 16), 17), (molecules.water_cluster(16, 16), 18),
                                    (molecules.water_cluster(24, 24), 26), (molecules.water_cluster(24, 24), 27),
                                    (molecules.water_cluster(25, 25), 32), (molecules.water_cluster(16, 16), 40)],
                         ids=lambda x: getattr(x, "name", str(x)))
def test_many_vectors_of_small_molecules(mol, k):
    """TDHF products of many vectors below 150 AOs take FP32 matrices: four chained sums of at most n rounded terms,
    sqrt(n) 2^-24 each."""
    print(f"[gpu] many vectors {mol.name} k={k}", flush=True)
    ctx = seqx.Context(0)
    ctx.set_params(*seqx.params_table(PR))
    job = ctx.prepare([mol.natoms], mol.Z, mol.xyz)
    n, o, v = job.dims()
    eps = job.scf_results()[0] / model.HARTREE_EV
    V = np.random.default_rng(5).normal(size=(k, o, v))
    diag = (eps[None, o:] - eps[:o, None]) * V
    ref = job.sigma(V, theory=seqx.TDHF)
    for precision in (seqx.FP32, seqx.BF16X3):
        for a, b in zip(job.sigma(V, theory=seqx.TDHF, precision=precision), ref):
            assert np.linalg.norm(a - b) <= 4 * np.sqrt(n) * 2.0 ** -24 * np.linalg.norm(b - diag)
    job.free()
    ctx.close()
