"""An image captured on a handle that holds the nodes of as many sample counts
as it keeps (16): a sample count among them is captured without a wait, and
every replay, with eager work between, equals the eager image bit for bit."""
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
            for rep in range(3):
                image.fill_(float("nan"))
                graph.replay()
                torch.randn(256, 256, device="cuda").matmul(torch.randn(256, 256, device="cuda"))
                stream.synchronize()
                assert torch.equal(image, ref[40]), rep
        finally:
            ctx.close()
