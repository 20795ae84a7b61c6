"""GPU: the no-allocation entry point keeps up with the device-tensor one.

Both take large P1 blocks by triangle pairs, the former with a smaller fixed
workspace; cut into many small panels such a block took two to four times as
long.  Fastest of several calls, entries against each other (two forms of the
same sums at most: FP64 1e-12, FP32 2e-6 of the largest entry) and, at some rows,
the oracle.
"""
import time

import numpy as np
import pytest

import oracle as O
from paper_1711_01897_amd import bem, inputs
from test_gpu_pairs import patch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("op", [bem.LAPLACE_SLP, bem.HELMHOLTZ_SLP])
@pytest.mark.parametrize("prec", [bem.FP32, bem.FP64])
def test_noalloc_time(op, prec):
    import torch
    xyz, tri = inputs.icosphere(5)
    mesh = bem.mesh_create(xyz, tri, 6)
    k = 5.0 if bem.is_complex(op) else 0.0
    rng = np.random.Generator(np.random.PCG64(8))
    rows, cols = patch(xyz, 3, 1023, rng), patch(xyz, 9000, 2049, rng)
    kind = torch.from_numpy(np.empty(0, dtype=bem.out_dtype(op, prec))).dtype
    outs = [torch.empty((1023, 2049), dtype=kind, device="cuda") for _ in range(2)]
    best = [1e9, 1e9]
    for _ in range(12):
        for i, fn in enumerate((bem.eval_entries_async, bem.eval_entries_async_noalloc)):
            torch.cuda.synchronize()
            t = time.perf_counter()
            fn(mesh, op, bem.P1, k, rows, cols, outs[i], prec=prec)
            torch.cuda.synchronize()
            best[i] = min(best[i], time.perf_counter() - t)
    a, b = (x.cpu().numpy() for x in outs)
    assert np.abs(a - b).max() <= (1e-12 if prec == bem.FP64 else 2e-6) * np.abs(a).max()
    some = rng.choice(1023, 3, replace=False)
    ref = O.OracleMesh(xyz, tri, 6).entries(op, O.P1, k, rows[some], cols, near=O.NEAR_SKIP)
    assert np.abs(b[some] - ref).max() <= (1e-11 if prec == bem.FP64 else 1e-4 if k else 1e-5) * np.abs(ref).max()
    assert best[1] <= 1.7 * best[0], best
    mesh.destroy()
