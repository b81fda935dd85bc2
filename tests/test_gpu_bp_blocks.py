"""Back-projection over blocks of voxels with a few frequency nodes each, and
on arrays of every block and step count (2, 4, 6 blocks of 16 Tx, 1 to 3 steps
of 32 Rx): the product engine against the Horner engine on every voxel and
against the FP64 oracle on sampled ones, relative to the image's peak (1e-4,
the engines' bar).  Grids of a few blocks with ragged edges, one voxel thick,
longer than a block along one axis only, coarse (every sample), and short
sweeps (K < 40: every sample); a cube of noise, whose image has no focus."""
import numpy as np
import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_tx,n_rx,K,dims,step", [
    (17, 33, 40, (9, 31, 30), 1e-3), (33, 65, 64, (25, 26, 51), 1e-3), (96, 96, 48, (24, 25, 23), 1e-3),
    (64, 32, 130, (1, 50, 7), 1e-3), (32, 64, 100, (50, 1, 1), 2e-3), (65, 31, 41, (2, 2, 2), 1e-3),
    (30, 37, 33, (7, 9, 11), 3e-3), (96, 65, 39, (5, 5, 5), 1e-3), (3, 2, 128, (40, 20, 20), 5e-4),
    (94, 94, 128, (6, 5, 4), 2e-2)])
def test_against_horner_and_oracle(gpu, orc, n_tx, n_rx, K, dims, step):
    import paper_2307_15412_amd as rr
    rng = np.random.default_rng(n_tx * 100 + n_rx)
    pos = lambda n: np.stack([np.zeros(n), rng.uniform(-0.07, 0.07, n), rng.uniform(-0.07, 0.07, n)], 1)
    array = sg.Array(pos(n_tx), pos(n_rx), 0.07, sg.MODE_SHARED).checked()
    chirp = sg.chirp_sfcw(n_steps=K)
    gpu.set_array(array.tx, array.rx, array.rx_radius, array.mode)
    gpu.set_chirp(chirp.f0, chirp.bandwidth, chirp.t_chirp, chirp.t_rep, K, 1)
    z = rng.standard_normal((n_tx * n_rx, 1, K, 2)).astype(np.float32)
    cube = torch.view_as_complex(torch.from_numpy(z)).cuda()
    grid = ((0.28, -step * dims[1] / 3, -step * dims[2] / 2), step, dims)
    got = gpu.backproject(cube, grid, engine=rr.GEMM_EXACT).reshape(-1)
    ref = gpu.backproject(cube, grid, engine=rr.DIRECT_FP32).reshape(-1)
    peak = float(ref.abs().max())
    assert float((got - ref).abs().max()) <= 1e-4 * peak
    assert torch.equal(gpu.backproject(cube, grid, engine=rr.ENGINE_AUTO).reshape(-1), got)
    sel = rng.choice(ref.numel(), min(6, ref.numel()), replace=False)
    i, j, k = np.unravel_index(sel, dims)
    vox = np.stack([grid[0][0] + i * step, grid[0][1] + j * step, grid[0][2] + k * step], -1)
    want = orc.backproject(array, chirp.f0, chirp.bandwidth / K, cube.cpu().numpy(), vox)
    assert np.abs(got[torch.from_numpy(sel).cuda()].cpu().numpy() - want).max() <= 1e-4 * peak
