"""GPU: dense assembly with many more rows than triangles.

Rows may repeat dofs and a panel of rows is cut by its distinct triangles, so
its rows are bounded apart from them: 300,000 rows of a few dofs, and 70,000
against more columns (whose panels' entries would otherwise be taken whole on
the device and in pinned memory), equal, bit for bit, the rows of the small matrix.
"""
import numpy as np
import pytest

import oracle as O
from paper_1711_01897_amd import bem, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,few,m,prec", [(300000, 12, 5, bem.FP32), (300001, 642, 3, bem.FP64), (70000, 40, 300, bem.FP32)])
def test_repeated_rows(n, few, m, prec):
    xyz, tri = inputs.icosphere(3)
    mesh = bem.mesh_create(xyz, tri, 4)
    rng = np.random.Generator(np.random.PCG64(6))
    dofs = rng.choice(len(xyz), few, replace=False).astype(np.int32)
    cols = rng.choice(len(xyz), m, replace=False).astype(np.int32)
    at = rng.integers(0, few, n)
    small = bem.eval_dense(mesh, bem.LAPLACE_SLP, bem.P1, 0.0, dofs, cols, prec=prec)
    ref = O.OracleMesh(xyz, tri, 4).entries(O.LAPLACE_SLP, O.P1, 0.0, dofs, cols, near=O.NEAR_SKIP)
    assert np.abs(small - ref).max() <= (1e-11 if prec == bem.FP64 else 1e-5) * np.abs(ref).max()
    got, st = bem.eval_dense(mesh, bem.LAPLACE_SLP, bem.P1, 0.0, dofs[at], cols, prec=prec, stats=True)
    assert np.array_equal(got, small[at])
    assert st["panels"] >= n / 65535
    mesh.destroy()
