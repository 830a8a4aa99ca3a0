"""The triangle's scan in double at the edges of its cell route: half-widths
whose knots (h, 2h, L - 2h) fall on cell boundaries, inside the first cell,
inside the last band (half the period) and on both sides of L/4, at particle
counts on both sides of the cell counts' steps, for spread and clustered
positions (every particle in one cell among them); against the oracle's direct
sums.

Tolerance: that of the triangle scan, 1e-12 of the objective and of the
objective term a pair sum enters: the cells hold exact offsets, and a band's
cubic carries a few rounding units of its terms."""
import math

import numpy as np
import pytest

import workloads as W
from tests.gpu_util import announce, host, to_gpu
from tests.test_gpu_triangle import check_cv, run_cv

pytestmark = pytest.mark.gpu


def cells(n):
    c = 256
    while c < 2048 and c * 16 < n:
        c *= 2
    return c


def edge_widths(n, L):
    C = cells(n)
    cell = L / C
    w = [0.3 * cell, 0.5 * cell, 0.75 * cell, cell, 1.25 * cell, 1.5 * cell, 2.0 * cell, 7.0 * cell, 7.5 * cell,
         0.25 * L - 0.6 * cell, 0.25 * L, 0.25 * L + 0.2 * cell, 0.25 * L + 0.5 * cell, 0.3 * L, 0.5 * L - 1.5 * cell,
         0.5 * L - cell, 0.5 * L - 0.6 * cell, 0.5 * L - 0.3 * cell, 0.5 * L]
    return np.array(w)


@pytest.mark.parametrize("kind", ["random", "even", "cluster", "one cell"])
@pytest.mark.parametrize("n", [2, 5, 255, 257, 1500, 4097])
def test_knots_on_and_between_cells(gpu, kind, n):
    L = 4.0
    rng = np.random.default_rng([53, n])
    if kind == "random":
        x = W.cosine_positions(rng, n, L, 0.4, 2 * math.pi / L)
    elif kind == "even":  # on the cells' boundaries where n divides the cells
        x = np.arange(n) / n * L
    elif kind == "cluster":
        x = np.concatenate([rng.normal(0.0, 0.01, n // 2), rng.normal(0.5 * L, 0.02, n - n // 2)]) % L
    else:
        x = 1.0 + 0.9 * (L / 2048) * rng.random(n)
    announce("tri cells", kind, n)
    widths = edge_widths(n, L)
    cv, sums, am = run_cv(gpu, x, L, widths, "f64")
    check_cv(cv, sums, am, x, L, widths, 1e-12)


def test_narrow_list_and_wrapped_input(gpu):
    """A list that reaches only a few bands, positions off [0, L)."""
    L, n = 2.75, 3000
    rng = np.random.default_rng(54)
    x = L * rng.random(n) + L * rng.integers(-3, 3, n)
    widths = np.geomspace(1e-4 * L, 0.02 * L, 9)
    announce("tri cells, narrow list")
    cv, sums, am = run_cv(gpu, x, L, widths, "f64")
    from oracle.vonmises import wrap
    check_cv(cv, sums, am, wrap(x, L), L, widths, 1e-12)


def test_non_finite_position_reaches_every_width(gpu):
    L = 4.0
    x = W.cosine_positions(np.random.default_rng(55), 700, L, 0.4, 2 * math.pi / L)
    x[33] = np.inf
    gpu.kde_numeric_check()
    announce("tri cells, non-finite")
    cv, sums, _ = run_cv(gpu, x, L, edge_widths(700, L), "f64")
    assert np.all(np.isnan(cv)) and np.all(np.isnan(sums))
    assert gpu.kde_numeric_check() == gpu.KDE_NUMERIC_POSITION
