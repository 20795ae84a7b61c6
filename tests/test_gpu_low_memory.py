"""GPU: little free device memory.

Device memory is filled up to a rest first.  What the library keeps between
calls (dense work areas, staging, pair workspaces) is given back when an
allocation of its own finds none, and a block whose triangle-pair workspace
cannot be had is taken by stars.
"""
import numpy as np
import pytest

import oracle as O
from paper_1711_01897_amd import bem, inputs
from test_gpu_pairs import patch, run

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def fill(rest):
    """Holds device memory until about `rest` bytes are left."""
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = lambda: torch.cuda.mem_get_info()[0]
    held = [torch.empty(free() - 4096 * MIB, dtype=torch.uint8, device="cuda")]
    while free() > rest + 32 * MIB:
        held.append(torch.empty(64 * MIB, dtype=torch.uint8, device="cuda"))
    return held


def drop(held):
    import torch
    held.clear()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


def test_server_starts_with_what_dense_assembly_kept():
    xyz, tri = inputs.icosphere(4)
    mesh = bem.mesh_create(xyz, tri, 4)
    every = np.arange(len(xyz), dtype=np.int32)
    want = bem.eval_dense(mesh, bem.LAPLACE_SLP, bem.P1, 0.0, every, every)   # keeps about 1 GiB
    bem.server_config(64 * MIB)
    bem.eval_entries(mesh, bem.LAPLACE_SLP, bem.P0, 0.0, every[:4], every)
    held = fill(768 * MIB)
    try:
        bem.server_config(1024 * MIB)
        got = bem.eval_entries(mesh, bem.LAPLACE_SLP, bem.P1, 0.0, every[:100], every)
    finally:
        drop(held)
        bem.server_config(1024 * MIB)
    assert np.abs(got - want[:100]).max() <= 2e-6 * np.abs(want).max()
    mesh.destroy()


def test_pair_block_without_workspace():
    xyz, tri = inputs.icosphere(5)
    mesh, om = bem.mesh_create(xyz, tri, 4), O.OracleMesh(xyz, tri, 4)
    rng = np.random.Generator(np.random.PCG64(7))
    rows, cols = patch(xyz, 7, 1500, rng), patch(xyz, 9000, 3000, rng)
    some = rng.choice(1500, 3, replace=False)
    ref = om.entries(O.LAPLACE_SLP, O.P1, 0.0, rows[some], cols, near=O.NEAR_SKIP)
    full = run(bem.eval_entries_async, mesh, bem.LAPLACE_SLP, bem.P1, 0.0, rows, cols, bem.FP32)
    mesh.destroy()                                  # the workspaces go with the last mesh
    mesh = bem.mesh_create(xyz, tri, 4)
    run(bem.eval_entries_async, mesh, bem.LAPLACE_SLP, bem.P1, 0.0, rows[:100], cols[:100], bem.FP32)
    import torch
    out = torch.empty((1500, 3000), device="cuda")
    held = fill(192 * MIB)                          # less than the block's 256 MiB
    try:
        bem.eval_entries_async(mesh, bem.LAPLACE_SLP, bem.P1, 0.0, rows, cols, out)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
    finally:
        drop(held)
    for m in (full, got):
        assert np.abs(m[some] - ref).max() <= 1e-5 * np.abs(ref).max()
    mesh.destroy()
