"""GPU: FP64 Helmholtz entries at wavenumbers whose phases a double does not resolve.

From k r = 2^51 pi on, r's rounding turns the phase by half a turn and more, so
the phase of an entry means nothing; but e^{ikr} keeps modulus one, so no entry
of the single layer (positive weights and basis functions) exceeds the Laplace
one in modulus.  Just below, at phases a double still resolves to a few thousandths,
the entries agree with the oracle to that.
"""
import numpy as np
import pytest

import oracle as O
from paper_1711_01897_amd import bem, inputs
from test_gpu_pairs import run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ico3():
    xyz, tri = inputs.icosphere(3)
    mesh = bem.mesh_create(xyz, tri, 6)
    yield xyz, tri, mesh, O.OracleMesh(xyz, tri, 6)
    mesh.destroy()


# row, star, triangle-pair, single-triangle and tiled forms
SHAPES = [(bem.P1, 3, 200), (bem.P1, 60, 100), (bem.P1, 300, 300), (bem.P0, 40, 300), (bem.P0, 1200, 1280)]


@pytest.mark.parametrize("k", [2.0 ** 50, 1e16, 1.2e18, 1e25, 1e100, 1e300])
def test_modulus_stays_one(ico3, k):
    xyz, tri, mesh, om = ico3
    rng = np.random.Generator(np.random.PCG64(9))
    for space, n, m in SHAPES:
        ndof = len(xyz) if space == bem.P1 else len(tri)
        rows, cols = rng.choice(ndof, n).astype(np.int32), rng.choice(ndof, m).astype(np.int32)
        lap = run(bem.eval_entries_async, mesh, bem.LAPLACE_SLP, space, 0.0, rows, cols, bem.FP64)
        got = run(bem.eval_entries_async, mesh, bem.HELMHOLTZ_SLP, space, k, rows, cols, bem.FP64)
        assert np.all(np.abs(got) <= lap * (1 + 1e-12)), (space, n, m)


def test_large_phases_still_resolved(ico3):
    xyz, tri, mesh, om = ico3
    rng = np.random.Generator(np.random.PCG64(10))
    k = 2.0 ** 40
    for space, n, m in SHAPES[:4]:
        ndof = len(xyz) if space == bem.P1 else len(tri)
        rows, cols = rng.choice(ndof, n).astype(np.int32), rng.choice(ndof, m).astype(np.int32)
        ref = om.entries(bem.HELMHOLTZ_SLP, space, k, rows, cols, near=O.NEAR_SKIP)
        lap = om.entries(bem.LAPLACE_SLP, space, 0.0, rows, cols, near=O.NEAR_SKIP)
        got = run(bem.eval_entries_async, mesh, bem.HELMHOLTZ_SLP, space, k, rows, cols, bem.FP64)
        # quadrature points of coordinates up to 1, three products each: 12 u in r on either side
        assert np.all(np.abs(got - ref) <= 24 * 2.0 ** -53 * k * lap)
