"""The node classes of the bands of path lengths (rr_bands.cpp, host code),
compiled for the CPU: for every class of a sample count, a unit path anywhere
within the class's reach is interpolated from the nodes to 2e-7 at every sample,
and the coefficients of a sample keep a 2-norm near one (1.25), so that
rounding in the node sums does not grow.  Sample counts at the edges of the
classes (five samples a node), primes, powers of two and long ones."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2307_15412_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "rr_internal.h"
int main(int argc, char **argv)
{
    for (int a = 1; a < argc; a++) {
        std::vector<int32_t> nodes;
        std::vector<float> coef;
        const int K = atoi(argv[a]);
        const BandClasses c = rr_band_classes(K, nodes, coef);
        const int32_t head[3] = {K, c.count, rr_band_nodes(K)};
        fwrite(head, 4, 3, stdout);
        for (int q = 0; q < c.count; q++) {
            fwrite(&c.n[q], 4, 1, stdout);
            fwrite(&c.z[q], 4, 1, stdout);
            fwrite(nodes.data() + q * RR_BAND_NMAX, 4, c.n[q], stdout);
            fwrite(coef.data() + c.coef[q], 4, (size_t)c.n[q] * K, stdout);
        }
    }
}
"""
COUNTS = [39, 40, 41, 59, 60, 61, 64, 79, 80, 97, 99, 100, 119, 120, 128, 139, 140, 159, 160, 161, 255, 256, 509,
          512, 1000, 1024, 1100]


@pytest.fixture(scope="module")
def classes(tmp_path_factory):
    d = tmp_path_factory.mktemp("bands")
    (d / "driver.cpp").write_text(DRIVER)
    exe = str(d / "driver")
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                    "-I" + os.path.join(ROOT, "include"), str(d / "driver.cpp"),
                    os.path.join(CSRC, "rr_bands.cpp"), "-o", exe], check=True)
    raw = subprocess.run([exe, *map(str, COUNTS)], check=True, capture_output=True).stdout
    out, at = {}, 0

    def take(dtype, n):
        nonlocal at
        v = np.frombuffer(raw, dtype, n, at)
        at += 4 * n
        return v

    for _ in COUNTS:
        K, count, most = take(np.int32, 3)
        cls = []
        for _ in range(count):
            n = int(take(np.int32, 1)[0])
            z = float(take(np.float32, 1)[0])
            cls.append((z, take(np.int32, n), take(np.float32, n * K).reshape(n, K)))
        out[int(K)] = (cls, int(most))
    assert at == len(raw)
    return out


@pytest.mark.parametrize("K", COUNTS)
def test_interpolation(classes, K):
    cls, most = classes[K]
    assert [len(r) for _, r, _ in cls] == [n for n in (8, 12, 16, 20, 24, 28, 32) if K >= 5 * n]
    assert most == (len(cls[-1][1]) if cls else 0)
    k = np.arange(K)
    for z, r, L in cls:
        assert r[0] == 0 and r[-1] == K - 1 and (np.diff(r) > 0).all()
        h = z / (np.pi * (K - 1))
        g = h * np.cos(np.linspace(0.0, np.pi, 201))
        want = np.exp(-2j * np.pi * np.outer(k, g))
        got = L.T.astype(np.float64) @ np.exp(-2j * np.pi * np.outer(r, g))
        assert np.abs(got - want).max() < 2e-7
        assert np.sqrt((L.astype(np.float64) ** 2).sum(0)).max() < 1.25
