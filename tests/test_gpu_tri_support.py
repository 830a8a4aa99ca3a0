"""The triangle's scan at the ends of a width's support: pairs at least h apart
add exactly 0 to S2 and pairs at least 2h apart (with their image, L - d)
exactly 0 to S1; no sum is negative, and a pair just inside adds what it should.

Separations are 1e-9 off the ends, far more than a position's rounding.
Tolerance inside: 1e-12 of a kernel's height, the scan's own."""
import numpy as np
import pytest

from oracle import triangle as tri
from tests.gpu_util import announce
from tests.test_gpu_triangle import run_cv

pytestmark = pytest.mark.gpu
EPS = 1e-9


def check(gpu, x, L, widths, dmin):
    """Particles whose smallest separation is dmin."""
    cv, sums, am = run_cv(gpu, x, L, widths, "f64")
    S1, S2 = sums[:len(widths)], sums[len(widths):]
    r1, r2 = tri.pair_sums(x, L, widths)
    assert np.all(S1 >= 0.0) and np.all(S2 >= 0.0)
    assert np.all(S2[widths <= dmin * (1 - EPS / 2)] == 0.0)
    assert np.all(S1[2 * widths <= dmin * (1 - EPS / 2)] == 0.0)
    assert np.all(np.abs(S1 - r1) <= 1e-12 * len(x) / widths) and np.all(np.abs(S2 - r2) <= 1e-12 * len(x) / widths)


@pytest.mark.parametrize("seed", range(24))
def test_two_particles(gpu, seed):
    L = 4.0
    rng = np.random.default_rng([57, seed])
    d = float(np.exp(rng.uniform(np.log(0.004), np.log(0.5)))) * L  # from about a cell to half the period
    x = np.array([rng.uniform(0, L - 1e-3), 0.0])
    x[1] = (x[0] + d) % L
    d = float(tri.periodic_distance(x[1] - x[0], L))
    w = [d * (1 - EPS) / 2, d * (1 + EPS) / 2, 0.7 * d, d * (1 - EPS), d * (1 + EPS), 1.2 * d, 2.3 * d,
         (L - d) / 2 * (1 - EPS), (L - d) / 2 * (1 + EPS), 0.3 * L, 0.5 * L]
    announce("tri support, two", seed, d)
    check(gpu, x, L, np.unique([h for h in w if h <= 0.5 * L]), d)


@pytest.mark.parametrize("n", [3, 40, 129, 600, 5000])
def test_evenly_spread_particles(gpu, n):
    L = 4.0
    gap = L / n
    x = (np.arange(n) + 0.37) * gap
    w = np.array([0.3, 0.5 - EPS, 0.5 + EPS, 0.8, 1 - EPS, 1 + EPS, 1.4, 1.5]) * gap
    announce("tri support, even", n)
    check(gpu, x, L, w[w <= 0.5 * L], gap)
