"""GPU: the server's kernel statistics count blocks by triangle pairs too."""
import numpy as np
import pytest

from paper_1711_01897_amd import bem, inputs
from test_gpu_pairs import patch

pytestmark = pytest.mark.gpu


def test_kernel_statistics_of_pair_blocks():
    xyz, tri = inputs.icosphere(4)
    mesh = bem.mesh_create(xyz, tri, 6)
    rng = np.random.Generator(np.random.PCG64(2))
    rows, cols = patch(xyz, 3, 700, rng), patch(xyz, 2000, 701, rng)
    ask = lambda: bem.eval_entries(mesh, bem.LAPLACE_DLP, bem.P1, 0.0, rows, cols, prec=bem.FP32, near=bem.NEAR_SKIP)
    ask()
    bem.server_stats(reset=True)
    bem.server_kernel_stats(reset=True)
    n = 24   # one batch in eight is timed
    for _ in range(n):
        ask()
    st, ks = bem.server_stats(), bem.server_kernel_stats()
    assert st["requests"] == n and st["entries"] == n * rows.size * cols.size
    assert st["kernel_launches"] >= 1 and st["kernel_seconds"] > 0
    assert st["kernel_seconds"] <= st["busy_seconds"]
    assert len(ks) == 1
    k = ks[0]
    assert (k["op"], k["space"], k["prec"], k["quad_points"]) == (bem.LAPLACE_DLP, bem.P1, bem.FP32, 6)
    timed = k["entries"] // (rows.size * cols.size)
    assert timed >= 2 and k["entries"] == timed * rows.size * cols.size
    assert k["pair_evals"] * n == st["kernel_evals"] * timed
    assert k["launches"] >= timed and k["workgroups"] > 0 and k["blocks"] > 0 and k["triangle_loads"] > 0
    assert 0 < k["seconds"] <= k["seconds_events"] * 1.001 + 1e-6
    mesh.destroy()
