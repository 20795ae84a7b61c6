"""GPU: P0 blocks by tiles of fixed triangles.

Blocks on both sides of the rule (2,048 workgroups) with every tile size,
remainders on both sides, either side fixed: the bits of the same entries
asked for in slices too small for tiles, and sampled rows against the FP64
oracle with the bounds of the entry tests (FP64 1e-11; FP32 1e-5 Laplace, 1e-4
Helmholtz, normwise).  Vertex-sharing pairs are skipped, refused or added as in
the slices.
"""
import numpy as np
import pytest

import oracle as O
from paper_1711_01897_amd import bem, inputs
from test_gpu_pairs import run

pytestmark = pytest.mark.gpu

OPS = [bem.LAPLACE_SLP, bem.LAPLACE_DLP, bem.LAPLACE_ADLP, bem.HELMHOLTZ_SLP, bem.HELMHOLTZ_DLP, bem.HELMHOLTZ_ADLP]


@pytest.fixture(scope="module")
def ico4():
    xyz, tri = inputs.icosphere(4)
    meshes = {q: (bem.mesh_create(xyz, tri, q), O.OracleMesh(xyz, tri, q)) for q in (4, 6)}
    yield len(tri), meshes
    for mesh, _ in meshes.values():
        mesh.destroy()


@pytest.mark.parametrize("op", OPS)
@pytest.mark.parametrize("prec", [bem.FP64, bem.FP32])
@pytest.mark.parametrize("q", [4, 6])
def test_tiles(ico4, op, prec, q):
    nt, meshes = ico4
    mesh, om = meshes[q]
    k = 6.0 if bem.is_complex(op) else 0.0
    rng = np.random.Generator(np.random.PCG64(9))
    # fixed triangles x lanes: workgroups with tiles of 1, 2, 4 and 8, the last tile short
    for n, m in ((204, 5120), (205, 5120), (411, 5119), (819, 4865), (1023, 4097)):
        a = rng.permutation(nt)[:n].astype(np.int32)
        b = rng.permutation(nt)[:m].astype(np.int32)
        for rows, cols in ((a, b), (b, a)):
            got = run(bem.eval_entries_async, mesh, op, bem.P0, k, rows, cols, prec)
            if rows is a:
                parts = [run(bem.eval_entries_async, mesh, op, bem.P0, k, rows[i:i + 100], cols, prec) for i in range(0, n, 100)]
                assert np.array_equal(got, np.concatenate(parts))
            else:
                parts = [run(bem.eval_entries_async, mesh, op, bem.P0, k, rows, cols[i:i + 100], prec) for i in range(0, n, 100)]
                assert np.array_equal(got, np.concatenate(parts, axis=1))
            some = np.array([0, len(rows) // 2, len(rows) - 1])
            ref = om.entries(op, O.P0, k, rows[some], cols, near=O.NEAR_SKIP)
            bound = 1e-11 if prec == bem.FP64 else (1e-4 if bem.is_complex(op) else 1e-5)
            assert np.abs(got[some] - ref).max() <= bound * np.abs(ref).max()


@pytest.mark.parametrize("prec", [bem.FP64, bem.FP32])
def test_touching_pairs(ico4, prec):
    nt, meshes = ico4
    mesh, _ = meshes[6]
    rng = np.random.Generator(np.random.PCG64(10))
    a, b = rng.permutation(nt)[:700].astype(np.int32), rng.permutation(nt)[:3000].astype(np.int32)
    got = run(bem.eval_entries_async, mesh, bem.LAPLACE_SLP, bem.P0, 0.0, a, b, prec, near=bem.NEAR_SINGULAR)
    parts = [run(bem.eval_entries_async, mesh, bem.LAPLACE_SLP, bem.P0, 0.0, a[i:i + 100], b, prec, near=bem.NEAR_SINGULAR)
             for i in range(0, 700, 100)]
    assert np.array_equal(got, np.concatenate(parts)) and np.all(got > 0)
    assert np.array_equal(bem.eval_entries(mesh, bem.LAPLACE_SLP, bem.P0, 0.0, a, b, prec=prec, near=bem.NEAR_SINGULAR), got)
    for fn in (bem.eval_entries_async, bem.eval_entries_async_noalloc):
        with pytest.raises(bem.BemError):
            run(fn, mesh, bem.LAPLACE_SLP, bem.P0, 0.0, a, b, prec, near=bem.NEAR_ERROR)
    with pytest.raises(bem.BemError):
        bem.eval_entries(mesh, bem.LAPLACE_SLP, bem.P0, 0.0, a, b, prec=prec, near=bem.NEAR_ERROR)
