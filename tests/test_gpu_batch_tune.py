"""The batch's autotuner against the engines it chooses from, on scenes of many
paths, whose engines a short prefix of the paths does not tell apart: the tuned
launch takes no more than the faster pinned engine's median plus a quarter and
50 us, and its counts and cubes are that scene's."""
import numpy as np
import pytest
import torch

import scenegen as sg
from helpers import rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shared,n_tx,n_rx,K,M,speed,rays", [
    (True, 32, 32, 128, 2, 0.0, 1_000_000), (True, 48, 64, 512, 1, 0.0, 1_000_000),
    (True, 20, 24, 96, 8, 2.0, 600_000), (False, 12, 16, 256, 8, 2.0, 600_000), (True, 4, 4, 64, 4, 0.0, 50_000)])
def test_tuned_is_the_faster(gpu, shared, n_tx, n_rx, K, M, speed, rays):
    import paper_2307_15412_amd as rr
    w = sg.workload_tiny(40)
    w.scene.obj_vel = np.array([[speed, 0.0, 0.0], [1.0, 0.0, 0.0]])
    w.array = sg.array_sparse_grid(n_tx, n_rx, 5, grid=128, mode=sg.MODE_SHARED if shared else sg.MODE_PER_TX)
    w.array.rx_radius = 1.0
    w.chirp = sg.Chirp(n_samples=K, n_chirps=M)
    w.trace.n_rays = rays
    B = rr.Batch(gpu, 1)
    B.set_workload(0, w)
    cubes = B.alloc_cubes()

    def median():
        B.launch(cubes)
        t = []
        for _ in range(7):
            B.launch(cubes)
            t.append(B.stats()["ms_total"])
        return float(np.median(t))

    pinned = {}
    for eng in (rr.DIRECT_FP32, rr.GEMM_EXACT):
        B.set_engine(0, eng)
        pinned[eng] = median()
    ref = cubes[0].clone()
    B.set_engine(0, rr.ENGINE_AUTO)
    B.tune(cubes)
    engine, tile = B.plan()
    tuned = median()
    print(f"direct {pinned[rr.DIRECT_FP32]:.3f} product {pinned[rr.GEMM_EXACT]:.3f} tuned {tuned:.3f} ms, "
          f"engine {engine[0]} tile {tile[0]}")
    assert rel_err(cubes[0].cpu().numpy(), ref.cpu().numpy()) < 1e-4
    assert tuned <= 1.25 * min(pinned.values()) + 0.05
    B.close()
