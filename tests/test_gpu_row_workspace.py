"""GPU: rows and columns with long lists at the limits of the workspaces.

The row form writes a block record for every 32 lane dofs, the star form one for
about a hundred, so a request near a limit (32 MiB of the no-allocation entry
point, a slot of the request server) can fit by stars alone.  It is taken that
way: entries against the FP64 oracle's small matrix (FP32 1e-5, FP64 1e-11 of the
largest entry), rows and columns.
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
    mesh, om = bem.mesh_create(xyz, tri, 4), O.OracleMesh(xyz, tri, 4)
    every = np.arange(len(xyz), dtype=np.int32)
    yield len(xyz), mesh, om.entries(O.LAPLACE_SLP, O.P1, 0.0, every, every, near=O.NEAR_SKIP)
    mesh.destroy()


def ask(ico3, n, m, prec, how, rows_fixed):
    nv, mesh, ref = ico3
    few = np.random.Generator(np.random.PCG64(4)).choice(nv, n, replace=False).astype(np.int32)
    many = np.sort(np.arange(m) % nv).astype(np.int32)   # repeated dofs lie together, as a mesh's order has neighbours
    rows, cols = (few, many) if rows_fixed else (many, few)
    if how == "noalloc":
        got = run(bem.eval_entries_async_noalloc, mesh, bem.LAPLACE_SLP, bem.P1, 0.0, rows, cols, prec)
    else:
        got = bem.eval_entries(mesh, bem.LAPLACE_SLP, bem.P1, 0.0, rows, cols, prec=prec, near=bem.NEAR_SKIP)
    limit = (1e-11 if prec == bem.FP64 else 1e-5) * np.abs(ref).max()
    assert np.abs(got - ref[rows][:, cols]).max() <= limit


@pytest.mark.parametrize("n,m,prec", [(64, 290000, bem.FP32), (16, 480000, bem.FP64)])
@pytest.mark.parametrize("rows_fixed", [True, False])
def test_noalloc(ico3, n, m, prec, rows_fixed):
    ask(ico3, n, m, prec, "noalloc", rows_fixed)


@pytest.mark.parametrize("n,m,prec", [(64, 190000, bem.FP32), (16, 330000, bem.FP64)])
@pytest.mark.parametrize("rows_fixed", [True, False])
def test_served(ico3, n, m, prec, rows_fixed):
    ask(ico3, n, m, prec, "served", rows_fixed)
