"""The refinement's Newton on both sides of its forms' lines: a bracket whose
series one wave holds in 128 or in 256 modes, a longer one by the workgroup
with its arrays in LDS, and a list long enough for them to be in the
workspace. The minimum is where the series, summed here in double with
scipy's Bessel functions, says it is.

Tolerance: 1e-12 of the sum of the objective's terms (a few hundred terms of
a rounding unit each, and scipy's own 1e-15); the concentration only to
1e-6, where a smooth minimum is flat."""
import math

import numpy as np
import pytest

from tests.gpu_util import announce, host, to_gpu

pytestmark = pytest.mark.gpu
L = 4 * math.pi


def objective(P, kappa, n):
    from scipy.special import ive
    m = np.arange(1, P.shape[0] + 1)
    rho = ive(m, kappa) / ive(0, kappa)
    a, c = rho * rho * P, rho * (P - n)
    scale = (2 * a.sum() / n**2 + 4 * np.abs(c).sum() / (n * (n - 1)) + 1) / L
    return (2 * a.sum() / n**2 - 4 * c.sum() / (n * (n - 1)) - 1) / L, scale


@pytest.mark.parametrize("sigma,k_hi", [(1.2, 1e3), (0.6, 1e4), (0.35, 1e4), (0.06, 5e5)])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_minimum_in_every_form(gpu, sigma, k_hi, dtype):
    n = 3001
    rng = np.random.default_rng([81, int(1000 * sigma)])
    x = ((2.0 + sigma * rng.standard_normal(n)) % L).astype(dtype)
    kap = np.exp(np.linspace(0, math.log(k_hi), 24))
    announce("refine", sigma, k_hi, dtype)
    res, cv, am = gpu.cv_refine(to_gpu(x), L, kap)
    res = host(res)
    assert 0 < int(host(am)[0]) < len(kap) - 1 and res[4] == host(am)[0]
    modes = int(12 * math.sqrt(kap[int(res[4]) + 1])) + 40
    th = 2 * math.pi * x.astype(np.float64) / L
    P = np.array([abs(np.exp(1j * m * th).sum())**2 for m in range(1, modes + 1)])
    f, scale = objective(P, res[0], n)
    assert abs(res[1] - f) <= 1e-12 * scale
    assert kap[int(res[4]) - 1] < res[0] < kap[int(res[4]) + 1]
    for side in (1 - 1e-3, 1 + 1e-3):
        assert objective(P, res[0] * side, n)[0] >= f - 1e-12 * scale
