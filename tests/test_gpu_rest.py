"""Paths at rest summed once (every engine): a path whose hits all lie on
resting objects adds the same to every chirp, so the records are split in two
parts before the sum.  Full cubes against the FP64 oracle with no, some, all
and all but one of the paths moving, per-element and shared launches, path
counts around the blocks of the split (1024) and above the moving count that
changes the layout (1024), one and several chirps, sample counts around the
direct engine's 16-sample runs; a batch slot equals the single-scene launch
bit for bit.  Bars: the engines' own (1e-4 direct and exact, 1e-3 for the
separable model's products)."""
import numpy as np
import pytest
import torch

import scenegen as sg
from helpers import oracle_to_soa, rel_err

pytestmark = pytest.mark.gpu


def _workload(mode, n_tx, n_rx, K, M, n_rays=150_000):
    w = sg.workload_tiny(5)
    w.scene.obj_vel = np.array([[0.0, 0.0, 0.0], [5.0, -2.0, 0.5]])
    w.array = (sg.array_sparse_grid(n_tx, n_rx, 3, mode=sg.MODE_SHARED) if mode == "shared"
               else sg.array_ula(n_tx, n_rx, mode=sg.MODE_PER_TX))
    w.chirp = sg.Chirp(n_samples=K, n_chirps=M)
    w.trace.n_rays = n_rays
    return w


def _moving(op, which, n_obj=2):
    """The oracle's path records with their ground hits given to the moving
    object (1) for the chosen paths, and every other hit to the ground."""
    op = op.copy()
    n = len(op)
    sel = {"none": np.zeros(n, bool), "some": np.random.default_rng(1).random(n) < 0.3,
           "all": np.ones(n, bool), "but_one": np.arange(n) != n // 2}[which]
    v = op["vid"]
    v[(v >= 0) & (v < n_obj)] = 0
    v[sel, 0] = 1
    op["vid"] = v
    return op


@pytest.mark.parametrize("which", ["none", "some", "all", "but_one"])
@pytest.mark.parametrize("mode,n_tx,n_rx,K,M,n", [("shared", 3, 5, 33, 3, 1025), ("shared", 20, 33, 16, 2, 1500),
                                                  ("per_tx", 4, 6, 65, 5, 1023), ("per_tx", 2, 3, 300, 2, 7),
                                                  ("shared", 2, 2, 17, 1, 1024)])
def test_every_engine(gpu, orc, mode, n_tx, n_rx, K, M, n, which):
    import paper_2307_15412_amd as rr
    w = _workload(mode, n_tx, n_rx, K, M)
    _, op = orc.trace(w.scene, w.array, w.trace, want_hits=False)
    assert len(op) >= n
    pick = np.sort(np.random.default_rng(2).choice(len(op), n, replace=False))
    op = _moving(op[pick], which)
    gpu.setup(w)
    gpu.set_paths({k: torch.from_numpy(np.ascontiguousarray(v)) for k, v in oracle_to_soa(op).items()})
    exact = orc.synth(op, w.scene, w.array, w.chirp, model=0)
    sep = orc.synth(op, w.scene, w.array, w.chirp, model=1)
    for model, engine, ref, tol in ((rr.EXACT, rr.DIRECT_FP32, exact, 1e-4), (rr.EXACT, rr.GEMM_EXACT, exact, 1e-4),
                                    (rr.SEPARABLE, rr.DIRECT_FP32, sep, 1e-4),
                                    (rr.SEPARABLE, rr.GEMM_BF16X3, sep, 1e-3)):
        got = gpu.synthesize(model=model, engine=engine).cpu().numpy()
        assert rel_err(got, ref) < tol, (model, engine)
    direct = gpu.synthesize(model=rr.EXACT, engine=rr.DIRECT_FP32)
    assert torch.equal(gpu.synthesize_noalloc(model=rr.EXACT), direct)
    idx = np.random.default_rng(3).choice(exact.size, min(64, exact.size), replace=False)
    got = gpu.synthesize(model=rr.EXACT, sample_idx=idx).cpu().numpy()
    assert rel_err(got, exact.reshape(-1)[idx]) < 1e-6


@pytest.mark.parametrize("mode,n_tx,n_rx,K,M", [("shared", 20, 33, 48, 4), ("per_tx", 3, 8, 128, 3),
                                                ("shared", 3, 4, 20, 1)])
@pytest.mark.parametrize("speed", [0.0, 3.0])
def test_batch_equals_single(gpu, mode, n_tx, n_rx, K, M, speed):
    """The moving ground makes every path a moving one."""
    import paper_2307_15412_amd as rr
    w = _workload(mode, n_tx, n_rx, K, M, 60_000)
    w.scene.obj_vel = np.array([[speed, 0.0, 0.0], [1.0, 0.0, 0.0]])
    for engine in (rr.DIRECT_FP32, rr.GEMM_EXACT):
        B = rr.Batch(gpu, 1)
        B.set_workload(0, w)
        B.set_engine(0, engine)
        cubes = B.alloc_cubes()
        counts = B.launch(cubes)
        gpu.setup(w)
        assert gpu.trace_workload(w, record_hits=False) == counts[0] > 1024
        ref = gpu.synthesize(model=rr.EXACT, engine=engine)
        assert torch.equal(cubes[0], ref), engine
        B.close()


@pytest.mark.parametrize("K", [1, 24, 54, 135, 195, 208])
def test_rest_as_exact_as_moving(gpu, orc, K):
    """The direct engine's chirp 0, the same paths at rest and moving (which
    are at the same place there): one run length of the rotations, so the same
    phasors; the resting sum adds them over the lanes, whose roundings are
    fewer than those of one lane's chain (a quarter more error is allowed for
    their chance)."""
    import paper_2307_15412_amd as rr
    w = _workload("shared", 3, 4, K, 2)
    _, op = orc.trace(w.scene, w.array, w.trace, want_hits=False)
    op = op[np.sort(np.random.default_rng(4).choice(len(op), 200, replace=False))]
    err = []
    for which in ("none", "all"):
        rec = _moving(op, which)
        gpu.setup(w)
        gpu.set_paths({k: torch.from_numpy(np.ascontiguousarray(v)) for k, v in oracle_to_soa(rec).items()})
        got = gpu.synthesize(model=rr.EXACT, engine=rr.DIRECT_FP32).cpu().numpy()[:, 0]
        ref = orc.synth(rec, w.scene, w.array, w.chirp, model=0)[:, 0]
        err.append(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    assert err[0] < 1.25 * err[1] < 1e-5, err


@pytest.mark.parametrize("mode,n_tx,n_rx,K", [("shared", 1, 1, 256), ("per_tx", 1, 4, 87), ("shared", 2, 2, 17),
                                              ("shared", 7, 8, 51), ("per_tx", 3, 85, 33), ("per_tx", 4, 64, 64)])
def test_rest_over_workgroups(gpu, orc, mode, n_tx, n_rx, K):
    """Samples of a channel over several workgroups, the last one short: few
    channels, as many as the compute units less one and as many; a batch slot
    equals the single-scene launch bit for bit.  Bar: the direct engine's."""
    import paper_2307_15412_amd as rr
    w = _workload(mode, n_tx, n_rx, K, 2, 20_000)
    gpu.setup(w)
    assert gpu.trace_workload(w, record_hits=False) > 0
    got = gpu.synthesize(model=rr.EXACT, engine=rr.DIRECT_FP32)
    _, op = orc.trace(w.scene, w.array, w.trace, want_hits=False)
    assert rel_err(got.cpu().numpy(), orc.synth(op, w.scene, w.array, w.chirp, model=0)) < 1e-4
    B = rr.Batch(gpu, 1)
    B.set_workload(0, w)
    B.set_engine(0, rr.DIRECT_FP32)
    cubes = B.alloc_cubes()
    B.launch(cubes)
    assert torch.equal(cubes[0], got)
    B.close()
