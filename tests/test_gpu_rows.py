"""GPU: P1 requests of few fixed dofs (eight threads per lane dof).

Every operator, precision and rule, both fixed sides, at the edges of a
workgroup's 32 vertices (256 discontinuous dofs), of the rule that takes the
form and of the one that shares a fixed star between waves, duplicated and shuffled dofs, a vertex in no triangle, and vertices whose
stars exceed eight triangles (a spheroid's poles), against the FP64 oracle with
the bounds of the star form (normwise FP64 1e-11; FP32 1e-5 Laplace, 1e-4
Helmholtz; the hypersingular operator in FP32 entrywise
8 u (1 + (r/h)^2) |ref| + 1e-6 max|ref|).
"""
import numpy as np
import pytest

import oracle as O
from paper_1711_01897_amd import bem, inputs
from test_gpu_pairs import OPS, check, run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mesh_of():
    """A spheroid with a fan of 24 triangles at vertex 0 and a vertex in no triangle."""
    ring = 24
    xyz, tri = inputs.spheroid(3.0, 1.0, 1500)
    phi = 2 * np.pi * np.arange(ring) / ring
    base = len(xyz)
    fan = np.vstack([[[8.0, 0.0, 0.0]], np.c_[np.full(ring, 8.2), np.cos(phi), np.sin(phi)], [[9.0, 9.0, 9.0]]])
    ftri = np.array([[base, base + 1 + i, base + 1 + (i + 1) % ring] for i in range(ring)], dtype=tri.dtype)
    xyz, tri = np.vstack([xyz, fan]), np.vstack([tri, ftri])
    meshes = {q: (bem.mesh_create(xyz, tri, q), O.OracleMesh(xyz, tri, q)) for q in (4, 6)}
    yield xyz, tri, base, meshes
    for mesh, _ in meshes.values():
        mesh.destroy()


@pytest.mark.parametrize("op", OPS)
@pytest.mark.parametrize("prec", [bem.FP64, bem.FP32])
@pytest.mark.parametrize("q", [4, 6])
def test_against_oracle(mesh_of, op, prec, q):
    xyz, tri, base, meshes = mesh_of
    mesh, om = meshes[q]
    k = 6.0 if bem.is_complex(op) else 0.0
    h = inputs.mean_edge_length(xyz, tri)
    rng = np.random.Generator(np.random.PCG64(7))
    every = len(xyz)
    for n, m in ((1, 1), (1, 31), (1, 32), (1, 33), (2, 97), (8, 64), (9, 65), (16, 1100), (17, 97), (64, 520),
                 (65, 97), (8, every), (8, 4100)):
        a = rng.choice(every, n).astype(np.int32)
        a[0] = base if n < 8 else every - 1      # the fan's centre; the vertex in no triangle
        b = (rng.choice(every, m) if m > every else rng.permutation(every)[:m]).astype(np.int32)
        if m > 32:
            b[[3, 32]] = base
        for rows, cols in ((a, b), (b, a)):
            ref = om.entries(op, O.P1, k, rows, cols, near=O.NEAR_SKIP)
            r = np.sqrt(((xyz[rows][:, None] - xyz[cols][None]) ** 2).sum(axis=2)) / h
            got = run(bem.eval_entries_async, mesh, op, bem.P1, k, rows, cols, prec)
            if np.abs(ref).max() > 0:
                check(got, ref, op, prec, r)
            else:
                assert np.all(got == 0)
            assert np.array_equal(bem.eval_entries(mesh, op, bem.P1, k, rows, cols, prec=prec, near=bem.NEAR_SKIP), got)
            assert np.array_equal(run(bem.eval_entries_async_noalloc, mesh, op, bem.P1, k, rows, cols, prec), got)


@pytest.mark.parametrize("prec", [bem.FP64, bem.FP32])
def test_discontinuous_singular_and_refused(mesh_of, prec):
    xyz, tri, base, meshes = mesh_of
    mesh, om = meshes[6]
    rng = np.random.Generator(np.random.PCG64(8))
    for op in OPS[:6]:
        k = 6.0 if bem.is_complex(op) else 0.0
        for n, m in ((1, 255), (3, 256), (8, 257), (2, 3 * len(tri))):
            a = rng.choice(3 * len(tri), n).astype(np.int32)
            b = rng.permutation(3 * len(tri))[:m].astype(np.int32)
            for rows, cols in ((a, b), (b, a)):
                got = run(bem.eval_entries_async, mesh, op, bem.DP1, k, rows, cols, prec)
                check(got, om.entries(op, O.DP1, k, rows, cols, near=O.NEAR_SKIP), op, prec, None)
    # singular pairs added to a row; a request whose triangles touch is refused, and only such a one
    op = bem.LAPLACE_SLP
    far = np.flatnonzero(xyz[:, 0] < -2.0).astype(np.int32)
    row = np.array([int(np.argmax(xyz[:base, 0]))], dtype=np.int32)
    star = np.unique(tri[np.any(tri == row[0], axis=1)])
    ring = np.setdiff1d(np.unique(tri[np.isin(tri, star).any(axis=1)]), star).astype(np.int32)
    full = run(bem.eval_entries_async, mesh, op, bem.P1, 0.0, row, ring, prec, near=bem.NEAR_SINGULAR)
    want = bem.eval_entries(mesh, op, bem.P1, 0.0, np.repeat(row, 12), ring, near=bem.NEAR_SINGULAR, prec=bem.FP64)[:1]
    assert ring.size > 8 and np.abs(full - want).max() <= (1e-12 if prec == bem.FP64 else 1e-5) * np.abs(want).max()
    run(bem.eval_entries_async, mesh, op, bem.P1, 0.0, row, far, prec, near=bem.NEAR_ERROR)
    for v in ring:
        cols = np.concatenate([far, [v]]).astype(np.int32)
        for rows_, cols_ in ((row, cols), (cols, row)):
            with pytest.raises(bem.BemError):
                run(bem.eval_entries_async, mesh, op, bem.P1, 0.0, rows_, cols_, prec, near=bem.NEAR_ERROR)
        with pytest.raises(bem.BemError):
            bem.eval_entries(mesh, op, bem.P1, 0.0, row, cols, prec=prec, near=bem.NEAR_ERROR)
