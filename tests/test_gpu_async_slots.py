"""GPU: the kept staging of eval_entries_async.

Far more calls in flight than there are slots (64), from two threads on two
streams each, of sizes that read the pinned image in place (up to 32
workgroups), that are copied, and that exceed a slot (8 MiB) and allocate
their own: every result bitwise that of the blocking call, whatever the slots
held before.  The slots go with the last mesh and come back with the next.
"""
import threading

import numpy as np
import pytest

from paper_1711_01897_amd import bem, inputs

pytestmark = pytest.mark.gpu


def requests(nv, nt):
    rng = np.random.Generator(np.random.PCG64(8))
    out = []
    for i in range(30):
        space, n = ((bem.P1, nv), (bem.P0, nt))[i % 2]
        nr, nc = ((1, 97), (33, 200), (300, 1), (257, 400), (2, 31 * 256))[i % 5]
        near = bem.NEAR_SINGULAR if i % 7 == 3 else bem.NEAR_SKIP
        out.append((bem.LAPLACE_SLP if i % 3 else bem.HELMHOLTZ_SLP, space, 0.0 if i % 3 else 3.0,
                    rng.integers(0, n, nr).astype(np.int32), rng.integers(0, n, nc).astype(np.int32),
                    (bem.FP32, bem.FP64)[i % 2], near))
    # past a slot: 300 x 3,000 P0 pairs of one triangle's neighbourhood repeated
    out.append((bem.LAPLACE_SLP, bem.P0, 0.0, np.zeros(300, dtype=np.int32), np.zeros(3000, dtype=np.int32), bem.FP32,
                bem.NEAR_SINGULAR))
    return out


def test_many_calls_in_flight():
    import torch
    kinds = {np.dtype(np.float32): torch.float32, np.dtype(np.float64): torch.float64,
             np.dtype(np.complex64): torch.complex64, np.dtype(np.complex128): torch.complex128}
    for level in (3, 2):   # the second mesh follows the end of the first
        xyz, tri = inputs.icosphere(level)
        mesh = bem.mesh_create(xyz, tri, 6)
        reqs = requests(xyz.shape[0], tri.shape[0])
        want = [bem.eval_entries(mesh, op, sp, k, r, c, prec=p, near=near) for op, sp, k, r, c, p, near in reqs]
        errors = []

        def caller(seed):
            try:
                torch.cuda.set_device(0)
                rng = np.random.Generator(np.random.PCG64(seed))
                streams = [torch.cuda.Stream(), torch.cuda.Stream()]
                got = []
                for j in range(160):
                    i = int(rng.integers(len(reqs) - 1)) if j % 40 else len(reqs) - 1
                    op, sp, k, r, c, p, near = reqs[i]
                    with torch.cuda.stream(streams[j % 2]):
                        out = torch.empty((r.size, c.size), dtype=kinds[want[i].dtype], device="cuda")
                    bem.eval_entries_async(mesh, op, sp, k, r, c, out, prec=p, near=near, stream=streams[j % 2])
                    got.append((i, out))
                torch.cuda.synchronize()
                for i, out in got:
                    if not np.array_equal(out.cpu().numpy(), want[i]):
                        errors.append(reqs[i][:3] + want[i].shape)
            except Exception as e:  # reported by the test's thread
                errors.append(e)

        threads = [threading.Thread(target=caller, args=(s,)) for s in (1, 2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not errors, errors[:3]
        mesh.destroy()
