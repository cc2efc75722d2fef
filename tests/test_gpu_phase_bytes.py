"""The bytes that the statistics count for the phases of a product, against the
stored form of each operand."""
import numpy as np
import pytest

from paper_2505_24807_amd import seqx
from synthetic import molecules, params

pytestmark = pytest.mark.gpu
PR = params.load()


# 90 AOs: matrices; 120: three planes; 96 occupied and 96 virtual orbitals or more, even numbers: two for the split
@pytest.mark.parametrize("mol, planes", [(molecules.water_cluster(15, 15), {seqx.FP64: 0, seqx.FP32: 0}),
                                         (molecules.water_cluster(20, 20), {seqx.FP32: 3, seqx.BF16X3: 3}),
                                         (molecules.water_cluster(67, 67), {seqx.FP32: 3, seqx.BF16X3: 2})],
                         ids=lambda x: getattr(x, "name", ""))
@pytest.mark.parametrize("theory", [seqx.CIS, seqx.TDHF])
def test_bytes_of_the_phases(mol, planes, theory):
    print(f"[gpu] phase bytes {mol.name} theory={theory}", flush=True)
    ctx = seqx.Context(0)
    ctx.set_params(*seqx.params_table(PR))
    for precision, p in planes.items():
        job = ctx.prepare([mol.natoms], mol.Z, mol.xyz)
        n, o, v = job.dims()
        k, pairs = 3, 12 * (mol.natoms // 3)
        nb = 2 * k if theory == seqx.TDHF else k
        job.sigma(np.ones((k, o, v)), theory=theory, precision=precision)
        d = 8 if precision == seqx.FP64 else 4

        def row(length, planes):  # blocks of 32 elements, two bytes a plane
            return -(-length // 32) * 64 * planes if planes else d * length

        c = 3 if p else 0
        expect = [n * row(o, c) + k * v * row(o, p) + k * n * row(v, p),
                  n * row(v, c) + k * n * row(v, p) + d * k * n * n,
                  d * k * n * n + nb * n * row(n, p) + 8 * pairs ** 2,
                  v * row(n, c) + nb * n * row(n, p) + nb * v * row(n, p),
                  o * row(n, c) + nb * v * row(n, p) + 16 * nb * o * v]
        assert list(job.stats().phase_bytes) == expect
        job.free()
    ctx.close()
