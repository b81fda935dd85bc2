"""An image captured on a handle that holds the nodes of 16 sample counts: one of
them is captured without a wait, and every replay equals the eager image bit
for bit, also after eager images of larger volumes and of other sample counts
on the same handle (the captured image's slices and node tables stay)."""
import numpy as np
import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu


def test_capture_among_sixteen():
    import paper_2307_15412_amd as rr
    rng = np.random.default_rng(1)
    pos = lambda n: np.stack([np.zeros(n), rng.uniform(-0.07, 0.07, n), rng.uniform(-0.07, 0.07, n)], 1)
    array = sg.Array(pos(20), pos(40), 0.07, sg.MODE_SHARED).checked()
    grid = ((0.28, -0.02, -0.02), 1e-3, (40, 41, 39))
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = rr.Context(0)
        try:
            ctx.set_array(array.tx, array.rx, array.rx_radius, array.mode)
            ref = {}
            for K in range(55, 39, -1):
                c = sg.chirp_sfcw(n_steps=K)
                ctx.set_chirp(c.f0, c.bandwidth, c.t_chirp, c.t_rep, K, 1)
                z = np.random.default_rng(K).standard_normal((800, 1, K, 2)).astype(np.float32)
                cube = torch.view_as_complex(torch.from_numpy(z)).cuda()
                ref[K] = ctx.backproject(cube, grid, engine=rr.GEMM_EXACT).clone()
            image = torch.empty_like(ref[40])
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
                ctx.backproject(cube, grid, out=image, engine=rr.GEMM_EXACT)
            for rep, (K, dims) in enumerate([(40, (50, 51, 49)), (40, (90, 80, 80)), (90, (60, 60, 60)),
                                             (57, (20, 20, 20)), (39, (30, 30, 30))]):
                c = sg.chirp_sfcw(n_steps=K)
                ctx.set_chirp(c.f0, c.bandwidth, c.t_chirp, c.t_rep, K, 1)
                other = torch.ones((800, 1, K), dtype=torch.complex64, device="cuda")
                ctx.backproject(other, (grid[0], 1e-3, dims), engine=rr.GEMM_EXACT)
                image.fill_(float("nan"))
                graph.replay()
                torch.randn(256, 256, device="cuda").matmul(torch.randn(256, 256, device="cuda"))
                stream.synchronize()
                assert torch.equal(image, ref[40]), rep
        finally:
            ctx.close()
