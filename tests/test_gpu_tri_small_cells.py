"""The triangle's scan in double with the cells that a sample of its size gets (8
to 2048): half-widths whose knots fall on, next to and
between the cells' boundaries, at particle counts on both sides of the counts'
steps, with the prefix moments' second places odd and even.

Tolerance: that of the triangle scan, 1e-12 of the objective and of the
objective term a pair sum enters."""
import math

import numpy as np
import pytest

import workloads as W
from tests.gpu_util import announce
from tests.test_gpu_triangle import check_cv, run_cv

pytestmark = pytest.mark.gpu


def cells(n):
    c = 256
    while c < 2048 and c * 16 < n:
        c *= 2
    while c > 8 and c * 8 >= n:
        c //= 2
    return c


@pytest.mark.parametrize("kind", ["random", "even", "one cell"])
@pytest.mark.parametrize("n", [2, 3, 31, 65, 128, 129, 1024, 1025, 2049, 6145])
def test_knots_about_the_cells(gpu, n, kind):
    L, C = 4.0, cells(n)
    cell = L / C
    rng = np.random.default_rng([58, n])
    if kind == "random":
        x = W.cosine_positions(rng, n, L, 0.4, 2 * math.pi / L)
    elif kind == "even":
        x = np.arange(n) / n * L
    else:
        x = 1.0 + 0.9 * cell * rng.random(n)
    w = np.array([0.01, 0.3, 0.5, 0.75, 1.0, 1.25, 1.5, 1.9, 2.0, 2.5, C / 4 - 0.6, C / 4, C / 4 + 0.2, C / 4 + 0.5,
                  0.3 * C, C / 3, C / 2 - 1.5, C / 2 - 1.0, C / 2 - 0.6, C / 2 - 0.3, C / 2]) * cell
    announce("tri small cells", n, kind)
    widths = np.unique(w[(w > 0) & (w <= 0.5 * L)])
    cv, sums, am = run_cv(gpu, x, L, widths, "f64")
    check_cv(cv, sums, am, x, L, widths, 1e-12)
    assert np.all(sums >= 0.0)


@pytest.mark.parametrize("sigma", [1e-5, 1e-3])
def test_few_cells_hold_the_sample(gpu, sigma):
    """Two clumps half a period apart, one of them about x = 0: widths narrower than
    a cell, inside a clump, between the clumps and half the period."""
    L, n = 4.0, 3000
    rng = np.random.default_rng([60, int(1e6 * sigma)])
    x = np.where(rng.random(n) < 0.7, sigma * L * rng.standard_normal(n), 0.5 * L * (1 + sigma * rng.standard_normal(n)))
    x = np.where(x % L >= L, 0.0, x % L)
    widths = np.array([0.02 * sigma, sigma, 3 * sigma, 0.1 / cells(n), 0.9 / cells(n), 0.01, 0.26, 0.4999, 0.5]) * L
    announce("tri small cells, clumps", sigma)
    cv, sums, am = run_cv(gpu, x, L, np.unique(widths), "f64")
    # the oracle gets the clump about 0 on one side of it, where its differences
    # are exact; of positions at both ends of the period its L - d carries their
    # rounding, which the narrowest width shows (1.2e-2 in S2 = 2.1e10)
    x = np.where(x > 0.75 * L, x - L, x)
    check_cv(cv, sums, am, x, L, np.unique(widths), 1e-12)
    assert np.all(sums >= 0.0)
