"""The smallest nodes of double deposits that the moments give (n M >= 2^25):
densities whose lowest node is 1/2 to 1/7 of the series' magnitude, against long
double sums over the particles.

Tolerance: 1e-15 relative per node. The series' rounding is about half a unit of
its magnitude (0.6 x 2.2e-16 x 7); the sum over the particles has 7e-16 itself."""
import math

import numpy as np
import pytest

import workloads as W
from tests.gpu_util import announce, host, to_gpu

pytestmark = pytest.mark.gpu
L, M, N = 4 * math.pi, 256, 1 << 17
LD = np.longdouble
PI = LD("3.14159265358979323846264338327950288")


def reference(x, kappa, nodes):
    theta = np.arange(4096).astype(LD) * (2 * PI / 4096)
    i0e = np.exp(LD(kappa) * (np.cos(theta) - 1)).mean()  # its trapezoidal sum is exact to e^-4000
    x, period = x.astype(LD), LD(L)
    out = []
    for g in nodes:
        s = np.sin((LD(g) * (period / M) - x) * (PI / period))
        out.append(np.exp(-2 * LD(kappa) * s * s).mean() / (period * i0e))
    return np.array(out)


@pytest.mark.parametrize("kappa", [2.0, 26.263635276533325, 144.0])
@pytest.mark.parametrize("amp", [0.5, 0.65, 0.75])
def test_lowest_nodes(gpu, amp, kappa):
    x = W.cosine_positions(np.random.default_rng([68, int(100 * amp)]), N, L, amp, 0.5)
    announce("deposit accuracy", amp, kappa)
    rho = host(gpu.deposit(to_gpu(x), L, M, kappa=kappa))
    nodes = np.unique(np.concatenate([np.argsort(rho)[:16], np.arange(0, M, 32)]))
    ref = reference(x, kappa, nodes)
    assert float(np.abs(rho[nodes] / ref - 1).max()) <= 1e-15


@pytest.mark.parametrize("kappa", [26.263635276533325, 144.0])
def test_clump_on_a_floor(gpu, kappa):
    rng = np.random.default_rng(69)
    k = N // 5
    x = np.concatenate([rng.random(N - k) * L, 0.3 * L + 0.02 * L * rng.standard_normal(k)]) % L
    x = np.where(x >= L, 0.0, x)
    announce("deposit accuracy, clump", kappa)
    rho = host(gpu.deposit(to_gpu(x), L, M, kappa=kappa))
    nodes = np.arange(1, M, 8)
    # (a node on the clump's flank carries the rounding of the sharp terms, 2e-15 over the particles)
    low = rho[nodes] < 1.5 * np.median(rho)
    ref = reference(x, kappa, nodes[low])
    assert float(np.abs(rho[nodes][low] / ref - 1).max()) <= 1e-15
