"""A captured trace (sync=False) replayed around eager work of the same handle:
a synthesis of more than 2^20 paths takes more pinned words than the trace made
room for, and the trace's own words must stay where the graph writes them.
Every replay gives the eager trace's count and paths bit for bit."""
import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu


def test_replay_after_large_synthesis():
    import paper_2307_15412_amd as rr
    w = sg.workload_tiny(3)
    w.array = sg.array_sparse_grid(1, 2, 3, mode=sg.MODE_SHARED)
    w.array.rx_radius = 1.0
    w.chirp = sg.Chirp(n_samples=2, n_chirps=2)
    w.trace.n_rays = 5_500_000
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = rr.Context(0)
        try:
            ctx.setup(w)
            n = ctx.trace_workload(w, record_hits=False)
            assert n > (1 << 20) + 2048
            ref = {k: v.clone() for k, v in ctx.paths().items()}
            ctx.trace_workload(w, record_hits=False, sync=False)
            assert ctx.path_count() == n
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
                ctx.trace_workload(w, record_hits=False, sync=False)
            first = None
            for rep in range(3):
                graph.replay()
                assert ctx.path_count() == n
                cube = ctx.synthesize(model=rr.EXACT, engine=rr.DIRECT_FP32).clone()
                torch.randn(256, 256, device="cuda").matmul(torch.randn(256, 256, device="cuda"))
                got = ctx.paths()
                assert all(torch.equal(got[k], ref[k]) for k in ref), rep
                first = cube if first is None else first
                assert torch.equal(cube, first), rep
            stream.synchronize()
        finally:
            ctx.close()
