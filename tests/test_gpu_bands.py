"""Bands of path lengths (tile layouts of the product engine): the sums of
resting paths from a few nodes per band must equal the FP64 oracle within the
engines' bars (1e-4 exact, 1e-3 separable): sample counts around the smallest
class (40 = 5 x 8) and several classes, ragged ones; path lists crowded into
one bin, spread over every class of width, spread thinner than a band takes
(48 paths), beyond the last band, and mixed; list sizes around the planning
blocks (4096) and the 32-path padding; repeated calls bit for bit, and a batch
slot equal to the single launch."""
import numpy as np
import pytest
import torch

import scenegen as sg
from helpers import oracle_to_soa, rel_err

pytestmark = pytest.mark.gpu


def _spread(op, how, rng, bin_m):
    """Move the oracle's hit points (K = 1 records) along their own direction
    so that the path lengths follow `how`."""
    op = op.copy()
    op["K"] = 1
    op["vid"][:, 0] = 0
    n = len(op)
    d = {"one_bin": rng.uniform(1.0, 1.0 + 0.2 * bin_m, n), "classes": rng.uniform(1.0, 1.0 + 12 * bin_m, n),
         "thin": rng.uniform(1.0, 1.0 + 200 * bin_m, n), "far": rng.uniform(1.0, 1.0 + 600 * bin_m, n)}
    d["mixed"] = np.where(np.arange(n) % 3 == 0, d["one_bin"], np.where(np.arange(n) % 3 == 1, d["classes"], d["far"]))
    q = rng.standard_normal((n, 3)) + np.array([3.0, 0.0, 0.0])
    q /= np.linalg.norm(q, axis=1, keepdims=True)
    op["p"][:, 0] = np.array([0.0, 0.0, 0.5]) + 0.5 * d[how][:, None] * q
    return op


@pytest.mark.parametrize("how", ["one_bin", "classes", "thin", "far", "mixed"])
@pytest.mark.parametrize("n_tx,n_rx,K,M,n", [(30, 40, 40, 1, 4097), (48, 20, 61, 2, 700), (31, 33, 131, 1, 4096),
                                             (29, 28, 200, 3, 33)])
def test_spread(gpu, orc, how, n_tx, n_rx, K, M, n):
    import paper_2307_15412_amd as rr
    w = sg.workload_tiny(9)
    w.array = sg.array_sparse_grid(n_tx, n_rx, 4, grid=128, mode=sg.MODE_SHARED)
    w.chirp = sg.Chirp(n_samples=K, n_chirps=M)
    w.trace.n_rays = 220_000
    _, op = orc.trace(w.scene, w.array, w.trace, want_hits=False)
    op = _spread(op[:n], how, np.random.default_rng(n), 299792458.0 / w.chirp.bandwidth)
    gpu.setup(w)
    gpu.set_paths({k: torch.from_numpy(np.ascontiguousarray(v)) for k, v in oracle_to_soa(op).items()})
    idx = np.random.default_rng(7).choice(n_tx * n_rx * M * K, 1500, replace=False)
    for model, engine, tol in ((rr.EXACT, rr.GEMM_EXACT, 1e-4), (rr.SEPARABLE, rr.GEMM_BF16X3, 1e-3)):
        cube = gpu.synthesize(model=model, engine=engine).clone()
        ref = orc.synth(op, w.scene, w.array, w.chirp, model=int(model), idx=idx)
        got = cube.reshape(-1)[torch.from_numpy(idx).cuda()].cpu().numpy()
        assert rel_err(got, ref) < tol, model
        direct = gpu.synthesize(model=model, engine=rr.DIRECT_FP32)
        assert rel_err(cube.cpu().numpy(), direct.cpu().numpy()) < tol, model
        assert torch.equal(gpu.synthesize(model=model, engine=engine), cube)


def test_batch_slot(gpu):
    import paper_2307_15412_amd as rr
    w = sg.Workload("hand", sg.scene_hand_proxy(3), sg.array_square(20), sg.chirp_sfcw(n_steps=64),
                    sg.TraceParams(n_rays=150_000, max_bounces=2, seed=3, az_min=-0.4, az_max=0.4, el_min=-0.4,
                                   el_max=0.4))
    B = rr.Batch(gpu, 1)
    B.set_workload(0, w)
    B.set_engine(0, rr.GEMM_EXACT)
    cubes = B.alloc_cubes()
    counts = B.launch(cubes)
    first = cubes[0].clone()
    B.launch(cubes)
    assert torch.equal(first, cubes[0])
    gpu.setup(w)
    assert gpu.trace_workload(w, record_hits=False) == counts[0] > 4096
    assert torch.equal(gpu.synthesize(model=rr.EXACT, engine=rr.GEMM_EXACT), first)
    B.close()
