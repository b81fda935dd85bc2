"""Product engine, paths at rest of arrays whose partial sums in bands would
take many times the cube: a 1024 x 1024 array takes every sample (19 GB of
partial sums at 40 samples beside a cube of 0.3 GB otherwise), a 256 x 256 one
with few paths the bands, with room for the bands that so few paths can fill.
Memory beside the cube, and the exact model's bar of 1e-4 against the FP64
oracle, one and several chirps."""
import numpy as np
import pytest
import torch

import scenegen as sg
from helpers import oracle_to_soa, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,K,M,n,bound", [(1024, 40, 1, 3000, 2 << 30), (1024, 40, 2, 100, 2 << 30),
                                              (256, 128, 1, 2000, 1 << 30)])
def test_partial_sums_bounded(orc, side, K, M, n, bound):
    import paper_2307_15412_amd as rr
    rng = np.random.default_rng(side + M)
    w = sg.workload_tiny(6)
    pos = np.array([0.0, 0.0, 0.5]) + np.stack([np.zeros(2 * side), rng.uniform(-0.2, 0.2, 2 * side),
                                                rng.uniform(-0.2, 0.2, 2 * side)], axis=1)
    w.array = sg.Array(pos[:side], pos[side:], 0.25, sg.MODE_SHARED).checked()
    w.chirp = sg.Chirp(n_samples=K, n_chirps=M)
    w.trace.n_rays = 250_000
    _, op = orc.trace(w.scene, w.array, w.trace, want_hits=False)
    op = op[:n]
    assert len(op) == n
    ctx = rr.Context(0)
    try:
        ctx.setup(w)
        ctx.set_paths({k: torch.from_numpy(np.ascontiguousarray(v)) for k, v in oracle_to_soa(op).items()})
        cube = torch.empty((side * side, M, K), dtype=torch.complex64, device="cuda:0")
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        ctx.synthesize(model=rr.EXACT, engine=rr.GEMM_EXACT, out=cube)
        torch.cuda.synchronize()
        assert free - torch.cuda.mem_get_info()[0] < bound
        idx = rng.choice(cube.numel(), 500, replace=False)
        ref = orc.synth(op, w.scene, w.array, w.chirp, model=0, idx=idx)
        got = cube.reshape(-1)[torch.from_numpy(idx).cuda()].cpu().numpy()
        assert rel_err(got, ref) < 1e-4
    finally:
        ctx.close()
