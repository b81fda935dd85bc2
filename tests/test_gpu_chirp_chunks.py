"""Product engine, more than 1024 moving paths on the Tx x Rx tiles with more
partial sums than one launch holds (128 MiB): the chirps go in chunks of ten,
the last one shorter.  Entries of the first, the boundary and the last chirps
against the FP64 oracle (1e-4, the engine's bar), and a batch slot equal to
the single launch bit for bit."""
import numpy as np
import pytest
import torch

import scenegen as sg
from helpers import rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [10, 13, 21])
def test_chunks(gpu, orc, M):
    import paper_2307_15412_amd as rr
    w = sg.workload_tiny(12)
    w.scene.obj_vel = np.array([[2.0, -1.0, 0.3], [0.0, 0.0, 0.0]])
    w.array = sg.array_sparse_grid(48, 64, 5, grid=128, mode=sg.MODE_SHARED)
    w.chirp = sg.Chirp(n_samples=512, n_chirps=M)
    w.trace.n_rays = 120_000
    gpu.setup(w)
    n = gpu.trace_workload(w, record_hits=False)
    _, op = orc.trace(w.scene, w.array, w.trace, want_hits=False)
    K = op["K"][:, None] > np.arange(op["vid"].shape[1])[None, :]
    assert n == len(op) and (K & (op["vid"] == 0)).any(axis=1).sum() > 1500
    cube = gpu.synthesize(model=rr.EXACT, engine=rr.GEMM_EXACT).clone()
    rng = np.random.default_rng(M)
    for m in sorted({0, 1, 9, min(10, M - 1), M - 2, M - 1}):
        c, k = rng.integers(0, 3072, 200), rng.integers(0, 512, 200)
        idx = (c * M + m) * 512 + k
        ref = orc.synth(op, w.scene, w.array, w.chirp, model=0, idx=idx)
        got = cube.reshape(-1)[torch.from_numpy(idx).cuda()].cpu().numpy()
        assert rel_err(got, ref) < 1e-4, m
    B = rr.Batch(gpu, 1)
    B.set_workload(0, w)
    B.set_engine(0, rr.GEMM_EXACT)
    cubes = B.alloc_cubes()
    for rep in range(2):
        cubes[0].fill_(float("nan"))
        assert B.launch(cubes)[0] == n
        assert torch.equal(cubes[0], cube), rep
    B.close()
