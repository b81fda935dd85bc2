"""Edges of the trace stage: ray counts around the tiles of the path-count
scan (256 rays), the coherent order's threshold (2^18 rays) and its
chunks, with and without recorded hits.  Paths must be bitwise the oracle's."""
import pytest

import scenegen as sg
from helpers import assert_paths_equal, gpu_soa_np, oracle_to_soa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_src", [1, 253, 254, 509, 4095, 4096, 87381, 87382, 262144])
@pytest.mark.parametrize("shared", [False, True])
def test_scan_and_order_edges(gpu, orc, per_src, shared):
    """Three sources (or one, shared) of per_src rays each and three point
    reflectors: the sources' virtual rays end on and beside tile bounds."""
    w = sg.workload_tiny(3)
    w.array = sg.array_sparse_grid(3, 4, 5, mode=sg.MODE_SHARED) if shared else sg.array_ula(3, 4)
    w.trace.n_rays = per_src if shared else 3 * per_src
    w.trace.max_bounces = 2
    _, op = orc.trace(w.scene, w.array, w.trace)
    o = oracle_to_soa(op)
    gpu.setup(w)
    for record in (True, False):
        assert gpu.trace_workload(w, record_hits=record) == len(op)
        assert_paths_equal(gpu_soa_np(gpu), o)
