"""Finite positions far beyond the period, whose wrap has no accuracy left: every
call reads its tables inside and returns; the other particles' results stay
what they are without them."""
import math

import numpy as np
import pytest

import workloads as W
from tests.gpu_util import announce, host, to_gpu

pytestmark = pytest.mark.gpu
L = 4 * math.pi


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n,M", [(3000, 64), (131072, 128), (131072, 256), (70000, 57)])
@pytest.mark.parametrize("shape", ["vm", "tri"])
def test_far_positions(gpu, dtype, n, M, shape):
    rng = np.random.default_rng([97, n, M])
    x = W.cosine_positions(rng, n, L, 0.3, 0.5).astype(dtype)
    far = rng.choice(n, 40, replace=False)
    big = np.array([1e17, -1e17, 1e20, -1e25, 1e30, -3e38])
    x[far] = big[np.arange(40) % 6].astype(dtype)
    near = np.setdiff1d(rng.choice(n, 300, replace=False), far)
    s = gpu.KDE_SHAPE_TRIANGLE if shape == "tri" else gpu.KDE_SHAPE_VONMISES
    k_i = np.full(n, 0.2 * L if shape == "tri" else 30.0, dtype=dtype)
    F = np.cos(np.arange(M) * (2 * math.pi / M)) + 1.5
    announce("far positions", dtype.__name__, n, M, shape)
    rho = host(gpu.deposit(to_gpu(x), L, M, kappa_i=to_gpu(k_i), shape=s))
    rho1 = host(gpu.deposit(to_gpu(x), L, M, kappa=float(k_i[0]), shape=s))
    assert np.all(np.isfinite(rho)) and np.all(rho >= 0) and np.all(np.isfinite(rho1)) and np.all(rho1 >= 0)
    out = host(gpu.gather(to_gpu(x), L, to_gpu(F), kappa_i=to_gpu(k_i), shape=s))
    assert np.all(np.isfinite(out))
    few = host(gpu.gather(to_gpu(x[near]), L, to_gpu(F), kappa_i=to_gpu(k_i[near]), shape=s))
    assert np.all(np.abs(out[near] - few) <= 1e-6 * few)
    if shape == "vm":
        w, lg, _ = gpu.adapt_widths(to_gpu(x), L, to_gpu(F), 20.0, 0.5)
        assert np.all(np.isfinite(host(w))) and np.isfinite(host(lg)[0])
        cv, _, _ = gpu.cv_scan(to_gpu(x[:3000]), L, [1.0, 30.0, 1e4])
        assert np.all(np.isfinite(host(cv)))
