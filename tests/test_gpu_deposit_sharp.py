"""The double deposit with one concentration at a call large enough for the
moments (n M >= 2^25): at the longest series their narrow form takes (order 112)
and the next one, and at concentrations far beyond any series, up to the
largest that the call accepts.

Against the oracle at sampled nodes (1e-12 relative, the deposit's own), or for
the sharpest kernels, whose terms hang on the last bit of a position, against
calls on parts of the particles, too small for the moments: each sums the same
positive terms in compensated runs, so 1e-13 is hundreds of their units."""
import math

import numpy as np
import pytest

import workloads as W
from oracle.vonmises import kernel
from tests.gpu_util import announce, host, rel_err, to_gpu

pytestmark = pytest.mark.gpu
L, M, N = 4 * math.pi, 256, 1 << 17


@pytest.mark.parametrize("kappa", [144.5, 145.0])
def test_longest_series_and_the_next(gpu, kappa):
    x = W.cosine_positions(np.random.default_rng(66), N, L, 0.4, 0.5)
    announce("deposit sharp", kappa)
    rho = host(gpu.deposit(to_gpu(x), L, M, kappa=kappa))
    nodes = np.arange(0, M, 15)
    ref = np.array([kernel(g * L / M - x, kappa, L).mean() for g in nodes])
    assert rel_err(rho[nodes], ref).max() <= 1e-12


@pytest.mark.parametrize("kappa", [1e6, 1e15, 1e17, 1e18, 1e33, 1e34, 1e100, 1e300])
def test_concentrations_beyond_any_series(gpu, kappa):
    x = W.cosine_positions(np.random.default_rng(67), N, L, 0.3, 0.5)
    x[::16] = (np.arange(N // 16) % (M - 3)) * (L / M)  # on nodes, all but the last three
    xt = to_gpu(x)
    announce("deposit sharp", kappa)
    rho = host(gpu.deposit(xt, L, M, kappa=kappa))
    part = N // 4
    ref = sum(host(gpu.deposit(xt[k * part:(k + 1) * part].clone(), L, M, kappa=kappa)) for k in range(4)) / 4
    assert ref[5] > 0.0 and np.all(np.isfinite(ref))
    assert np.all(np.abs(rho - ref) <= 1e-13 * ref)
