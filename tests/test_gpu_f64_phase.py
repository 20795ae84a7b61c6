"""GPU: the FP64 kernels' own e^{ikr} and reciprocal square root.

Phases from far below a half turn to 1e5 radians (several thousand half
turns), for both rules and every Helmholtz operator form, against the FP64
oracle.  The oracle rounds k r once before its sine and cosine, which moves
its phase by up to k r 2^-53; the bound is twice that on top of 1e-13 of the
largest entry (36 terms of a few ulps each).  The double layer and the
hypersingular operator scale with k r and (k r)^2 like their entries do.
"""
import numpy as np
import pytest

import oracle as O
from paper_1711_01897_amd import bem, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1e-3, 0.7, 31.0, 1.0e3, 5.0e4])
@pytest.mark.parametrize("q", [4, 6])
def test_phase_against_oracle(k, q):
    xyz, tri = inputs.icosphere(2)
    mesh = bem.mesh_create(xyz, tri, q)
    om = O.OracleMesh(xyz, tri, q)
    bound = 1e-13 + 2.0 * (2.0 * k) * 2.0 ** -53
    try:
        for op in (bem.HELMHOLTZ_SLP, bem.HELMHOLTZ_DLP):
            for space, n in ((bem.P0, tri.shape[0]), (bem.P1, xyz.shape[0])):
                rows, cols = np.arange(3, 36, dtype=np.int32), np.arange(n - 70, n, dtype=np.int32)
                ref = om.entries(op, space, k, rows, cols, near=O.NEAR_SKIP)
                for r, c, want in ((rows, cols, ref), (cols, rows, om.entries(op, space, k, cols, rows,
                                                                               near=O.NEAR_SKIP))):
                    got = bem.eval_entries(mesh, op, space, k, r, c, prec=bem.FP64)
                    assert np.max(np.abs(got - want)) <= bound * np.max(np.abs(want)), (op, space, k, q)
    finally:
        mesh.destroy()


def test_coincident_points_stay_infinite():
    """Two triangles on the same place that share no vertex index: every point
    meets its copy at distance zero, and the entry is infinite."""
    xyz, tri = inputs.icosphere(0)
    xyz2, tri2 = np.vstack([xyz, xyz]), np.vstack([tri, tri + xyz.shape[0]]).astype(np.int32)
    mesh = bem.mesh_create(xyz2, tri2, 6)
    try:
        got = bem.eval_entries(mesh, bem.LAPLACE_SLP, bem.P0, 0.0, [0], [20, 21, 13], prec=bem.FP64)
        assert np.isposinf(got[0, 0]) and np.all(np.isfinite(got[0, 1:]))
    finally:
        mesh.destroy()
