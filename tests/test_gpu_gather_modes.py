"""The double gather through the field's modes (n M >= 2^25 and the grids and
concentrations its rule names) against the sum over the nodes: orders below
and above M/2, M and the highest mode taken, concentrations from 0 past what
the series serves, in one call, fields with empty stretches, and non-finite
inputs.

Tolerance: a value of the series is at least 1/256 of its magnitude, whose
rounding is a few dozen units, so 2e-12 of the value; a value summed over the
nodes carries some units of the sum of magnitudes, 1e-13 of it."""
import math

import numpy as np
import pytest

import workloads as W
from oracle.vonmises import kernel, wrap
from tests.gpu_util import announce, host, to_gpu

pytestmark = pytest.mark.gpu
L = 4 * math.pi


def check(gpu, out, x, kap, F, M, sample):
    """Against the oracle; concentrations above 2000, where the rounding of
    the wrapped position alone moves a term by sqrt(kappa) units, against the
    same particles in a call small enough for the sum over the nodes."""
    nodes = np.arange(M) * (L / M)
    few = host(gpu.gather(to_gpu(x[sample]), L, to_gpu(F), kappa_i=to_gpu(kap[sample])))
    for k, i in enumerate(sample):
        K = kernel(nodes - wrap(x[i], L), kap[i], L) * (L / M)
        ref, mag = float((F * K).sum()), float((np.abs(F) * K).sum())
        ref = few[k] if kap[i] > 2000 else ref
        assert abs(out[i] - ref) <= 2e-12 * abs(ref) + 1e-13 * mag, (i, x[i], kap[i], out[i], ref)


def field(kind, M, rng):
    th = np.arange(M) * (2 * math.pi / M)
    if kind == "modes":
        return np.sin(th + 0.3) + 0.4 * np.cos(3 * th) + 0.05 * rng.standard_normal(M)
    if kind == "density":  # empty but for a clump
        return np.exp(-0.5 * ((th - 1.0) / 0.05) ** 2)
    F = np.zeros(M)
    F[M // 3] = 1.0
    return F


@pytest.mark.parametrize("kind", ["modes", "density", "one node"])
@pytest.mark.parametrize("n,M", [(131072, 256), (131073, 257), (300001, 256), (800001, 300), (32768, 4096)])
def test_per_particle_concentrations(gpu, n, M, kind):
    rng = np.random.default_rng([71, n, M])
    x = rng.uniform(-L, 2 * L, n)
    kap = 10.0 ** rng.uniform(0.0, 2.5, n)
    special = np.array([0.0, 1e-300, 1e-30, 1e-12, 1e-3, 700.0, 2000.0, 2400.0, 2.0e4, 1e7, 1e15])
    at = rng.choice(n, 4 * len(special), replace=False)
    kap[at] = np.repeat(special, 4)
    kap[: n // 8] = np.minimum(kap[: n // 8], 20.0)  # workgroups of low order
    F = field(kind, M, rng)
    announce("gather modes", n, M, kind)
    out = host(gpu.gather(to_gpu(x), L, to_gpu(F), kappa_i=to_gpu(kap)))
    check(gpu, out, x, kap, F, M, np.concatenate([at, rng.choice(n, 150, replace=False), [0, n - 1]]))


@pytest.mark.parametrize("kappa", [0.0, 1e-15, 3.0, 120.0, 150.0, 3000.0])
@pytest.mark.parametrize("n,M", [(600000, 64), (262145, 128)])
def test_one_concentration(gpu, n, M, kappa):
    rng = np.random.default_rng([72, M])
    x = W.cosine_positions(rng, n, L, 0.4, 0.5)
    F = field("modes", M, rng)
    announce("gather modes", n, M, kappa)
    out = host(gpu.gather(to_gpu(x), L, to_gpu(F), kappa=kappa))
    check(gpu, out, x, np.full(n, kappa), F, M, rng.choice(n, 100, replace=False))


def test_non_finite_inputs(gpu):
    n, M = 131072, 256
    rng = np.random.default_rng(73)
    x, kap = rng.uniform(0, L, n), np.full(n, 30.0)
    F = field("modes", M, rng)
    bad_x, bad_k = [5, 70000], [9, 131071]
    xb, kb = x.copy(), kap.copy()
    xb[bad_x] = [np.nan, np.inf]
    kb[bad_k] = [np.nan, np.inf]
    gpu.kde_numeric_check()
    announce("gather modes, non-finite particles")
    out = host(gpu.gather(to_gpu(xb), L, to_gpu(F), kappa_i=to_gpu(kb)))
    assert gpu.kde_numeric_check() == gpu.KDE_NUMERIC_POSITION | gpu.KDE_NUMERIC_CONCENTRATION
    assert np.all(np.isnan(out[bad_x]))
    good = np.setdiff1d(rng.choice(n, 100, replace=False), bad_x + bad_k)
    check(gpu, out, x, kap, F, M, good)
    # a field with an infinite node: every particle is summed over the nodes
    F[7] = np.inf
    announce("gather modes, infinite field")
    assert np.all(host(gpu.gather(to_gpu(x), L, to_gpu(F), kappa_i=to_gpu(kap))) == np.inf)
