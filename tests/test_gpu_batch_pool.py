"""A batch whose rays return more paths than the pool it starts with (65 536):
the launch that overflows reads none of the pool's unwritten places (its paths
count as none until the pool has grown), and the cubes and counts it returns
after the re-run equal the single launches bit for bit, at rest and moving, on
the direct engine, the product engine's bands and its sample split."""
import numpy as np
import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu


def _workload(i, shared, n_tx, n_rx, K, M, rays, speed):
    w = sg.workload_tiny(30 + i)
    w.scene.obj_vel = np.array([[speed, 0.0, 0.0], [1.0, 0.0, 0.0]])
    mode = sg.MODE_SHARED if shared else sg.MODE_PER_TX
    w.array = sg.array_sparse_grid(n_tx, n_rx, 2 + i, mode=mode)
    w.array.rx_radius = 1.0        # a fifth of the rays pass so wide a sphere
    w.chirp = sg.Chirp(n_samples=K, n_chirps=M)
    w.trace.n_rays = rays
    return w


SCENES = [(True, 20, 18, 64, 2, 250_000, 0.0), (False, 3, 4, 48, 2, 150_000, 0.0),
          (True, 17, 33, 40, 2, 60_000, 2.0), (True, 4, 4, 32, 3, 80_000, 2.0)]


@pytest.mark.parametrize("engine", ["direct", "product"])
def test_pool_overflow(gpu, engine):
    import paper_2307_15412_amd as rr
    eng = rr.DIRECT_FP32 if engine == "direct" else rr.GEMM_EXACT
    ws = [_workload(i, *a) for i, a in enumerate(SCENES)]
    refs = []
    for w in ws:
        gpu.setup(w)
        n = gpu.trace_workload(w, record_hits=False)
        refs.append((n, gpu.synthesize(model=rr.EXACT, engine=eng).clone()))
    assert sum(n for n, _ in refs) > 1.25 * 65536
    B = rr.Batch(gpu, len(ws))
    for i, w in enumerate(ws):
        B.set_workload(i, w)
        B.set_engine(i, eng)
    cubes = B.alloc_cubes()
    for rep in range(3):
        for c in cubes:
            c.fill_(float("nan"))
        counts = B.launch(cubes)
        for i, (n, ref) in enumerate(refs):
            assert counts[i] == n, (rep, i)
            assert torch.equal(cubes[i], ref), (rep, i)
    B.close()
