"""The exact pilot's widths on both sides of the line between one and four
particles per thread, with remainders and with several Horner runs: ratios of
the widths against the oracle's density at sampled particles, and the
geometric mean, which the widths' own logarithms have to give back.

Tolerance: 1e-12 in double (a hundred modes of a rounding unit, a logarithm
and an exponential), two float units on top in float."""
import math

import numpy as np
import pytest

import workloads as W
from oracle.vonmises import kernel
from tests.gpu_util import announce, host, to_gpu

pytestmark = pytest.mark.gpu
L = 4 * math.pi


@pytest.mark.parametrize("n", [524287, 524289, 600001])
@pytest.mark.parametrize("kappa", [3.0, 500.0])
@pytest.mark.parametrize("dtype,tol", [("float64", 1e-12), ("float32", 2.4e-7)])
def test_widths(gpu, n, kappa, dtype, tol):
    rng = np.random.default_rng([91, n])
    x = W.cosine_positions(rng, n, L, 0.4, 0.5).astype(dtype)
    announce("exact widths", n, kappa, dtype)
    k_i, log_g, floored = gpu.adapt_widths_exact(to_gpu(x), L, kappa, 0.5)
    k_i = host(k_i).astype(np.float64)
    assert int(host(floored)[0]) == 0
    assert abs(np.log(k_i).mean() - math.log(kappa)) <= tol
    at = np.concatenate([[0, n - 1], rng.choice(n, 6, replace=False)])
    xd = x.astype(np.float64)
    f = np.array([kernel(xd[i] - xd, kappa, L).mean() for i in at])
    want = kappa * f / math.exp(float(host(log_g)[0]))
    assert np.abs(k_i[at] / want - 1.0).max() <= tol
