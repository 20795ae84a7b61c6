"""GPU: blocks by triangle pairs through the request server, up to a slot's size.

A request's entries lie once in the slot's host staging and once, with the local
matrices, in its device arena.  Blocks whose entries take from a third of a
slot to nearly all of it (default arena: 64 MiB slots; 4 MiB arena: 1 MiB ones)
are served as they were by single stars: against the device-tensor request (two
forms of the same sums: FP64 1e-12, FP32 2e-6 of the largest entry) and, at some
rows, the oracle (FP64 1e-11, FP32 1e-5 Laplace, 1e-4 Helmholtz).
"""
import numpy as np
import pytest

import oracle as O
from paper_1711_01897_amd import bem, inputs
from test_gpu_pairs import patch, run

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def served(level, n, m, op, k, prec, q=6):
    xyz, tri = inputs.icosphere(level)
    mesh = bem.mesh_create(xyz, tri, q)
    rng = np.random.Generator(np.random.PCG64(5))
    rows, cols = patch(xyz, 7, n, rng), patch(xyz, len(xyz) - 9, m, rng)
    got = bem.eval_entries(mesh, op, bem.P1, k, rows, cols, prec=prec, near=bem.NEAR_SKIP)
    again = bem.submit(mesh, op, bem.P1, k, rows, cols, prec=prec, near=bem.NEAR_SKIP).wait()
    assert np.array_equal(got, again)
    dev = run(bem.eval_entries_async, mesh, op, bem.P1, k, rows, cols, prec)
    assert np.abs(got - dev).max() <= (1e-12 if prec == bem.FP64 else 2e-6) * np.abs(dev).max()
    some = rng.choice(n, 3, replace=False)
    ref = O.OracleMesh(xyz, tri, q).entries(op, O.P1, k, rows[some], cols, near=O.NEAR_SKIP)
    limit = 1e-11 if prec == bem.FP64 else (1e-4 if bem.is_complex(op) else 1e-5)
    assert np.abs(got[some] - ref).max() <= limit * np.abs(ref).max()
    mesh.destroy()


@pytest.mark.parametrize("level,n,m,op,k,prec", [
    (4, 2562, 2562, bem.LAPLACE_SLP, 0.0, bem.FP32),      # 25 MiB of entries
    (4, 2562, 2562, bem.HELMHOLTZ_SLP, 3.0, bem.FP32),    # 50
    (4, 2562, 2562, bem.LAPLACE_DLP, 0.0, bem.FP64),      # 50
    (5, 1024, 4096, bem.LAPLACE_SLP, 0.0, bem.FP64),      # 32
    (4, 2000, 2000, bem.LAPLACE_ADLP, 0.0, bem.FP64),     # 31
    (5, 1600, 6100, bem.LAPLACE_SLP, 0.0, bem.FP32),     # 37
])
def test_default_arena(level, n, m, op, k, prec):
    served(level, n, m, op, k, prec)


@pytest.mark.parametrize("n,op,prec", [(300, bem.LAPLACE_SLP, bem.FP64), (300, bem.LAPLACE_HYPS, bem.FP64),
                                       (360, bem.LAPLACE_SLP, bem.FP32), (300, bem.HELMHOLTZ_DLP, bem.FP32)])
def test_small_slots(n, op, prec):
    bem.server_config(4 * MIB)
    try:
        served(3, n, n, op, 3.0 if bem.is_complex(op) else 0.0, prec)
    finally:
        bem.server_config(1024 * MIB)
