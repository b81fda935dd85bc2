"""Back-projection on the matrix cores: every leg is the correctly rounded FP64
length rounded once to FP32, voxel by voxel.  One transmitter, one receiver and
one sample (every-sample path), the cube's only entry 1: a voxel's value is
the product of two phasors whose phases are the FP32 products of the rounded
legs with f / c, formed here in the same arithmetic.  Bar: the split operands'
2^-16 and the hardware sin/cos (2e-6 rad at the most) add up below 3e-5; a leg one
FP32 unit off at 0.5 to 1 m turns the phase by 9e-5 rad at 72 GHz.  Legs within
1e-15 of the middle between two FP32 numbers are left out (the FP64 roundings
of the two sides may differ there)."""
import numpy as np
import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu


def test_legs_rounded_once(gpu):
    import paper_2307_15412_amd as rr
    dims, step, origin = (192, 512, 512), 4.1e-4, (0.55, -0.105, -0.105)
    el = np.array([[0.0, 0.0137, -0.0071], [0.0, -0.0093, 0.0111]])
    chirp = sg.chirp_sfcw(n_steps=2)
    gpu.set_array(el[:1], el[1:], 0.07, sg.MODE_SHARED)
    gpu.set_chirp(chirp.f0, 0.0, chirp.t_chirp, chirp.t_rep, 1, 1)
    cube = torch.ones((1, 1, 1), dtype=torch.complex64, device="cuda:0")
    got = gpu.backproject(cube, (origin, step, dims), engine=rr.GEMM_EXACT)
    fc = float(np.float32(chirp.f0 * (1.0 / 299792458.0)))
    axes = [origin[a] + torch.arange(dims[a], dtype=torch.float64, device="cuda:0") * step for a in range(3)]
    worst = 0.0
    for i in range(0, dims[0], 16):
        x, y, z = torch.meshgrid(axes[0][i:i + 16], axes[1], axes[2], indexing="ij")
        turns, sure = torch.zeros_like(x), torch.ones_like(x, dtype=torch.bool)
        for e in el:
            d = torch.sqrt((x - e[0]) ** 2 + (y - e[1]) ** 2 + (z - e[2]) ** 2)
            u = d * 2.0 ** 24                         # 0.5 <= d < 1: FP32 units
            sure &= (u - torch.floor(u) - 0.5).abs() > 2.0 ** 24 * 1e-15
            turns += (d.float().double() * fc).float().double()
        want = torch.polar(torch.ones_like(turns), 2.0 * np.pi * (turns - torch.round(turns)))
        off = (got[i:i + 16].to(torch.complex128) - want).abs()
        worst = max(worst, float(off[sure].max()))
    assert worst < 3e-5, worst
