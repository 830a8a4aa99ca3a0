"""The double gather through the field's modes (n M >= 2^25): its error against
long double sums over the nodes, for fields that change sign, lie low over a part
of the period or over most of it; and fields scaled by powers of two far up
and down, which scale every value by the same power, bit for bit.

Tolerance: 6e-15 of sum |F_g| K_i per particle: a value's local size is at
least 1/16 of the series', whose rounding is about half a unit (16 x 1.1e-16 x
3 for the largest of thousands); a sum over the nodes has about half of that.
To it comes what a rounding unit of the particle's phase does, 2.2e-16 sum |F_g|
|dK_i / dtheta| (3e-15 of the magnitudes at concentrations of some hundreds, in
a sum over the nodes as well: 8.2e-15 at the worst particle of these)."""
import math

import numpy as np
import pytest

from tests.gpu_util import announce, host, to_gpu

pytestmark = pytest.mark.gpu
L, N = 4 * math.pi, 1 << 17
LD = np.longdouble
PI = LD("3.14159265358979323846264338327950288")


def field(kind, M, rng):
    th = np.arange(M) * (2 * math.pi / M)
    if kind == "modes":
        F = 0.05 * rng.standard_normal(M)
        for m in range(1, 5):
            F += (rng.standard_normal() * np.cos(m * th) + rng.standard_normal() * np.sin(m * th)) / m
        return F
    if kind == "low":
        return 1.0 + 0.95 * np.cos(th)
    return 0.01 + np.exp(-0.5 * ((th - 1.0) / 0.3) ** 2)  # "bump"


def reference(x, kap, F):
    """The sums, their magnitudes' and those of their slopes' magnitudes, per
    particle, at the position's rounded fraction of the period."""
    M = len(F)
    c1 = np.cos(np.arange(2048).astype(LD) * (2 * PI / 2048)) - 1
    g = np.arange(M).astype(LD) / M
    out = []
    for f, k in zip((x / L).astype(LD), kap.astype(LD)):
        K = np.exp(-2 * k * np.sin((g - f) * PI) ** 2) / np.exp(k * c1).mean() / M
        slope = k * np.abs(np.sin(2 * PI * (g - f))) * K
        out.append(((F * K).sum(), (np.abs(F) * K).sum(), (np.abs(F) * slope).sum()))
    return np.array(out).T


@pytest.mark.parametrize("M,k_lo,k_hi", [(256, 14.0, 68.0), (256, 200.0, 800.0), (512, 2.0, 20.0)])
@pytest.mark.parametrize("kind", ["modes", "low", "bump"])
def test_error_against_long_double(gpu, kind, M, k_lo, k_hi):
    rng = np.random.default_rng([75, M, int(k_hi)])
    x = rng.random(N) * L
    kap = np.exp(rng.uniform(math.log(k_lo), math.log(k_hi), N))
    F = field(kind, M, rng)
    announce("gather accuracy", kind, M, k_lo)
    out = host(gpu.gather(to_gpu(x), L, to_gpu(F), kappa_i=to_gpu(kap)))
    at = rng.choice(N, 1500, replace=False)
    ref, mag, slope = reference(x[at], kap[at], F)
    err = np.abs(out[at].astype(LD) - ref)
    assert np.all(err <= 6e-15 * mag + 2.2e-16 * slope)
    assert float(np.sqrt((err ** 2).sum() / (ref ** 2).sum())) <= 6e-16


@pytest.mark.parametrize("power", [-900, -520, 330, 900])
@pytest.mark.parametrize("kind", ["modes", "bump"])
def test_scaled_fields(gpu, kind, power):
    M = 256
    rng = np.random.default_rng(76)
    x = rng.random(N) * L
    kap = np.exp(rng.uniform(math.log(1.0), math.log(1000.0), N))
    kap[:: 7] = 0.0
    kap[1:: 7] = 10.0 ** rng.uniform(-300.0, -3.0, len(kap[1:: 7]))
    F = field(kind, M, rng)
    announce("gather scaled", kind, power)
    one = host(gpu.gather(to_gpu(x), L, to_gpu(F), kappa_i=to_gpu(kap)))
    out = host(gpu.gather(to_gpu(x), L, to_gpu(np.ldexp(F, power)), kappa_i=to_gpu(kap)))
    assert np.all(np.isfinite(out)) and np.array_equal(out, np.ldexp(one, power))
