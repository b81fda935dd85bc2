"""Fused backward pass and weight gradients: how the rows are split over
workgroups (128-row steps, at most 256 workgroups) at the sizes where the
split changes, against an FP64 network whose hidden activations are rounded
to FP16 as the kernels round them."""
import numpy as np
import pytest
import torch

from oracle import mlp

pytestmark = pytest.mark.gpu


def _round(x):
    return np.asarray(x, dtype=np.float32).astype(np.float16).astype(np.float64)


def _rounded_grad(params, codes, hist):
    p = mlp.unpack(_round(params))
    X = mlp.features(_round(codes))
    h1 = _round(np.maximum(X @ p["W1"].T + p["b1"], 0.0))
    h2 = _round(np.maximum(h1 @ p["W2"].T + p["b2"], 0.0))
    h3 = _round(np.maximum(h2 @ p["W3"].T + p["b3"], 0.0))
    z = (h3 @ p["W4"].T + p["b4"]).reshape(len(hist), -1)
    e = np.exp(z - z.max(1, keepdims=True))
    dz = ((e / e.sum(1, keepdims=True) - hist / hist.sum(1, keepdims=True)) / len(hist)).reshape(-1)
    d3 = dz[:, None] * p["W4"] * (h3 > 0)
    d2 = (d3 @ p["W3"]) * (h2 > 0)
    d1 = (d2 @ p["W2"]) * (h1 > 0)
    g = {"W1": d1.T @ X, "b1": d1.sum(0), "W2": d2.T @ h1, "b2": d2.sum(0), "W3": d3.T @ h2,
         "b3": d3.sum(0), "W4": dz[None] @ h3, "b4": dz.sum()[None]}
    return np.concatenate([np.ravel(g[k]) for k, _ in mlp.SHAPES])


@pytest.mark.parametrize("S", [1, 4, 5, 33])
def test_gradient_split(gpu, S):
    """64, 256, 320 (two steps a workgroup) and 2112 steps (nine, the last
    workgroup short).  Rounding every activation to FP16 moves these gradients
    by up to 4 % of their norm; an FP32 sum rounds one activation in about
    7000 (1e-7 of 7e-4) otherwise than FP64 does, so sqrt(1 / 7000) of that,
    5e-4, is to be expected, and 5e-3 is ten times as much.  One wrong row
    block of S * 64 steps would change the gradient by more."""
    rng = np.random.default_rng(100 + S)
    codes = (rng.random((S, 16)) * (rng.random((S, 16)) < 0.4)).astype(np.float32)
    hist = (rng.random((S, 8192)) * (rng.random((S, 8192)) < 0.03)).astype(np.float32)
    gpu.mlp_init(6)
    _, g = gpu.mlp_train_step(torch.from_numpy(codes).cuda(), torch.from_numpy(hist).cuda(), 0.0,
                              want_grad=True)
    ref = _rounded_grad(gpu.mlp_get_params(), codes, hist.astype(np.float64))
    g = g.cpu().numpy().astype(np.float64)
    rel = np.linalg.norm(g - ref) / np.linalg.norm(ref)
    print(f"gradient vs rounded FP64 network ({S} scenes): {rel:.2e}")
    assert rel < 5e-3
