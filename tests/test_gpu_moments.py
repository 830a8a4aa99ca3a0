"""The Fourier moments at the edges of their kernel's forms, against the
oracle's direct pair sums: series orders on both sides of the narrow form's
last mode (112), of the wide form's tiles (232, 480 and 728 modes: four, two
and one waves per tile) and of its mode blocks (976 modes), and particle
counts around a wave's group (64), a team's pair of groups (128) and a
workgroup's (512).

Tolerance: that of the Fourier scan (1e-12 of each objective value and pair
sum, and 1e-13 of the double sum a pair sum is the difference of): a phase is
at most 7 rotations, about 10 rounding units, from one reduced exactly."""
import math

import numpy as np
import pytest

import workloads as W
from oracle import cv as ocv
from oracle.vonmises import conv2_at_zero, kernel
from tests.gpu_util import announce, host, rel_err, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 63, 65, 128, 129, 511, 513, 1100])
@pytest.mark.parametrize("top", [0.3, 130.0, 160.0, 600.0, 700.0, 2600.0, 2900.0, 6200.0, 6700.0, 11000.0, 12000.0,
                                 5e4, 1e6])
def test_orders_and_counts_at_the_kernel_edges(gpu, n, top):
    L = 4 * math.pi
    x = W.cosine_positions(np.random.default_rng([41, n]), n, L, 0.4, 0.5)
    kap = np.array([0.02, 0.1, 0.5, 1.0]) * top
    announce("moments", n, top)
    cv, sums, _ = gpu.cv_scan_fourier(to_gpu(x), L, kap)
    cv, sums = host(cv), host(sums)
    ref_cv, S1, S2 = ocv.cv_curve(x, L, kap)
    assert rel_err(cv, ref_cv).max() <= 1e-12
    tot1 = n * conv2_at_zero(kap, L) + 2 * S1
    tot2 = n * kernel(0.0, kap, L) + 2 * S2
    assert np.all(np.abs(sums[:4] - S1) <= 1e-12 * np.abs(S1) + 1e-13 * tot1)
    assert np.all(np.abs(sums[4:] - S2) <= 1e-12 * np.abs(S2) + 1e-13 * tot2)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [40000, 140001])
def test_chunks_of_several_groups(gpu, dtype, n):
    """Counts whose chunks hold several groups per team, with an odd number
    of groups in the last, and positions outside [0, L)."""
    L = 2.75
    rng = np.random.default_rng([43, n])
    x = L * rng.random(n) + L * rng.integers(-2, 3, n)
    x = x.astype(np.float64 if dtype == "f64" else np.float32)
    kap = np.array([1.0, 30.0, 400.0, 4000.0])
    announce("moments of several groups", dtype, n)
    cv, sums, _ = gpu.cv_scan_fourier(to_gpu(x), L, kap)
    from oracle.vonmises import wrap
    ref_cv, S1, S2 = ocv.cv_curve_fourier(wrap(x.astype(np.float64), L), L, kap)
    assert rel_err(host(cv), ref_cv).max() <= 1e-12
    assert rel_err(host(sums)[:4], S1).max() <= 1e-12 and rel_err(host(sums)[4:], S2).max() <= 1e-12
