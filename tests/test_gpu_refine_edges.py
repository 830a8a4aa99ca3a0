"""The refinement where its bracket ends at a concentration whose series is one
mode longer at exp(log(kappa)) than at kappa (M^2 + 40 kappa a perfect square,
M the order): by the workgroup with its arrays in LDS.

Tolerance: 1e-12 of the sum of the objective's terms, as for the other forms."""
import math

import numpy as np
import pytest

from tests.gpu_util import announce, host, to_gpu
from tests.test_gpu_refine_forms import objective

pytestmark = pytest.mark.gpu
L = 4 * math.pi


@pytest.mark.parametrize("k_hi", [3678.0, 4455.0, 4726.0, 5005.0])
def test_bracket_ends_on_a_perfect_square(gpu, k_hi):
    n = 3001
    rng = np.random.default_rng(83)
    x = (2.0 + 0.02 * rng.standard_normal(n)) % L  # sharper than the list: its last concentration is the best
    kap = np.concatenate([np.geomspace(1.0, 3000.0, 7), [k_hi]])
    announce("refine edges", k_hi)
    res, cv, am = gpu.cv_refine(to_gpu(x), L, kap)
    res = host(res)
    assert int(host(am)[0]) == len(kap) - 1 == int(res[4]) and res[0] == k_hi
    th = 2 * math.pi * x / L
    P = np.array([abs(np.exp(1j * m * th).sum())**2 for m in range(1, int(12 * math.sqrt(k_hi)) + 40)])
    f, scale = objective(P, k_hi, n)
    assert abs(res[1] - f) <= 1e-12 * scale and abs(host(cv)[-1] - f) <= 1e-12 * scale
