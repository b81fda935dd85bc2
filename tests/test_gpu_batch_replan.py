"""A batch scene left to AUTO whose leg tables pass the budget by its rays (1 in
16) and fit it by the first launch's count: the second launch, into new cubes,
moves it to the product engine and computes its cube (captured anew), as does
every launch after it."""
import pytest
import torch

import scenegen as sg
from helpers import rel_err

pytestmark = pytest.mark.gpu


def test_new_cubes_after_the_first_count(gpu):
    import paper_2307_15412_amd as rr
    w = sg.workload_tiny(50)
    w.array = sg.array_sparse_grid(48, 64, 5, grid=128, mode=sg.MODE_SHARED)
    w.chirp = sg.Chirp(n_samples=64, n_chirps=256)
    w.trace.n_rays = 1_400_000
    B = rr.Batch(gpu, 1)
    B.set_workload(0, w)
    cubes = B.alloc_cubes()
    n = B.launch(cubes)[0]
    assert B.plan()[0][0] == rr.DIRECT_FP32
    ref = cubes[0].cpu().numpy()
    for rep in range(3):
        other = B.alloc_cubes()
        other[0].fill_(float("nan"))
        assert B.launch(other)[0] == n
        assert rel_err(other[0].cpu().numpy(), ref) < 1e-4, rep
    assert B.plan()[0][0] == rr.GEMM_EXACT
    B.close()
