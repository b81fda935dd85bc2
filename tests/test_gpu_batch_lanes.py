"""A batch whose product-engine scenes run side by side: every replay of the
captured launch, with other work in between, gives each scene's single-launch
cube bit for bit, whatever lane its scene is in, and whether its rays are
traced in coherent order (4096 rays a source or more) or as drawn."""
import numpy as np
import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu


def _workload(i, shared, n_tx, n_rx, K, M, rays):
    w = sg.workload_tiny(20 + i)
    w.array = sg.array_sparse_grid(n_tx, n_rx, 3 + i, mode=sg.MODE_SHARED if shared else sg.MODE_PER_TX)
    w.chirp = sg.Chirp(n_samples=K, n_chirps=M)
    w.trace.n_rays = rays
    return w


SCENES = [(True, 17, 20, 64, 3, 60_000), (False, 4, 12, 96, 2, 50_000), (True, 33, 8, 40, 1, 3_000),
          (False, 3, 16, 128, 4, 9_000), (True, 5, 4, 32, 2, 200_000), (False, 6, 6, 64, 2, 30_000)]


@pytest.mark.parametrize("n_exact", [1, 2, 6])
def test_lanes_replay(gpu, n_exact):
    import paper_2307_15412_amd as rr
    ws = [_workload(i, *a) for i, a in enumerate(SCENES)]
    eng = [rr.GEMM_EXACT if i < n_exact else rr.DIRECT_FP32 for i in range(len(ws))]
    refs = []
    for w, e in zip(ws, eng):
        gpu.setup(w)
        n = gpu.trace_workload(w, record_hits=False)
        refs.append((n, gpu.synthesize(model=rr.EXACT, engine=e).clone()))
    B = rr.Batch(gpu, len(ws))
    for i, w in enumerate(ws):
        B.set_workload(i, w)
        B.set_engine(i, eng[i])
    cubes = B.alloc_cubes()
    for rep in range(3):
        for c in cubes:
            c.fill_(float("nan"))
        counts = B.launch(cubes)
        torch.randn(512, 512, device="cuda").matmul(torch.randn(512, 512, device="cuda"))
        for i, (n, ref) in enumerate(refs):
            assert counts[i] == n, (rep, i)
            assert torch.equal(cubes[i], ref), (rep, i)
    B.close()
