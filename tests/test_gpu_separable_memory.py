"""Separable model, a small array (which the GEMM pads to 256 channels) and many
moving paths over many chirps: the leg tables of the product engine would take
tens of GB, so the moving paths run as the GEMM, whose operands take a
fraction, and the cube holds the engine's bar of 1e-3 against the FP64 oracle."""
import numpy as np
import pytest
import torch

import scenegen as sg
from helpers import oracle_to_soa, rel_err

pytestmark = pytest.mark.gpu


def test_moving_tables_within_budget(orc):
    import paper_2307_15412_amd as rr
    n = 300_000
    w = sg.workload_tiny(6)
    w.scene.obj_vel = np.array([[4.0, -1.0, 0.0], [5.0, -2.0, 0.5]])
    w.array = sg.array_sparse_grid(1, 60, 3, mode=sg.MODE_SHARED)
    w.chirp = sg.Chirp(n_samples=256, n_chirps=256)
    w.trace.n_rays = 100_000
    _, op = orc.trace(w.scene, w.array, w.trace, want_hits=False)
    op = np.tile(op, -(-n // len(op)))[:n]
    op["amp"] *= np.random.default_rng(1).uniform(0.5, 1.5, n)
    ctx = rr.Context(0)
    try:
        ctx.setup(w)
        ctx.set_paths({k: torch.from_numpy(np.ascontiguousarray(v)) for k, v in oracle_to_soa(op).items()})
        cube = torch.empty((60, 256, 256), dtype=torch.complex64, device="cuda:0")
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        ctx.synthesize(model=rr.SEPARABLE, engine=rr.GEMM_BF16X3, out=cube)
        torch.cuda.synchronize()
        assert free - torch.cuda.mem_get_info()[0] < 8 << 30
        idx = np.random.default_rng(7).choice(cube.numel(), 300, replace=False)
        ref = orc.synth(op, w.scene, w.array, w.chirp, model=1, idx=idx)
        got = cube.reshape(-1)[torch.from_numpy(idx).cuda()].cpu().numpy()
        assert rel_err(got, ref) < 1e-3
    finally:
        ctx.close()
