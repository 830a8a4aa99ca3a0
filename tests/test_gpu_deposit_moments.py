"""The double pilot deposit through the moments (n M >= 2^25 and a series that
fits the narrow form): against the sum over the particles at sampled nodes,
on both sides of each of its rules, and the batched engine with the same bits.
Where the density has empty stretches the grid has to come from the sum over
the particles, which keeps the relative accuracy of its smallest nodes.

Tolerance: 1e-12 relative per node, the deposit's own (a node is at least an
eighth of the series' magnitude, so it carries a few dozen rounding units)."""
import math

import numpy as np
import pytest

import workloads as W
from oracle.vonmises import kernel
from tests.gpu_util import announce, host, rel_err, to_gpu

pytestmark = pytest.mark.gpu


def reference(x, kappa, M, L, nodes):
    return np.array([kernel(g * L / M - x, kappa, L).mean() for g in nodes])


@pytest.mark.parametrize("n,M", [(1 << 17, 256), ((1 << 17) - 1, 256), (140001, 300), (8192, 4096), (600001, 57)])
@pytest.mark.parametrize("kappa", [0.0, 0.3, 26.3, 145.0, 147.0])
def test_both_sides_of_the_rules(gpu, n, M, kappa):
    L = 4 * math.pi
    x = W.cosine_positions(np.random.default_rng([61, n]), n, L, 0.5, 0.5)
    announce("deposit moments", n, M, kappa)
    rho = host(gpu.deposit(to_gpu(x), L, M, kappa=kappa))
    nodes = np.unique(np.linspace(0, M - 1, 9).astype(int))
    assert rel_err(rho[nodes], reference(x, kappa, M, L, nodes)).max() <= 1e-12


@pytest.mark.parametrize("kind", ["cluster", "one point", "off period"])
def test_grids_the_series_does_not_serve(gpu, kind):
    L, M, n, kappa = 4 * math.pi, 256, 1 << 17, 60.0
    rng = np.random.default_rng(62)
    if kind == "cluster":
        x = rng.normal(0.3 * L, 0.02 * L, n) % L
    elif kind == "one point":
        x = np.full(n, 0.7 * L)
    else:
        x = L * rng.random(n) + L * rng.integers(-2, 3, n)
    announce("deposit moments", kind)
    rho = host(gpu.deposit(to_gpu(x), L, M, kappa=kappa))
    nodes = np.arange(0, M, 31)
    from oracle.vonmises import wrap
    assert rel_err(rho[nodes], reference(wrap(x, L), kappa, M, L, nodes)).max() <= 1e-12


def test_non_finite_position_makes_every_node_nan(gpu):
    L, M, n = 4 * math.pi, 256, 1 << 17
    x = W.cosine_positions(np.random.default_rng(63), n, L, 0.3, 0.5)
    x[777] = np.nan
    gpu.kde_numeric_check()
    announce("deposit moments, non-finite")
    assert np.all(np.isnan(host(gpu.deposit(to_gpu(x), L, M, kappa=20.0))))
    assert gpu.kde_numeric_check() == gpu.KDE_NUMERIC_POSITION


def test_batch_gives_the_same_bits(gpu):
    """A set whose pilot comes from the moments, one with an empty stretch
    (the sum over the particles follows) and a small one, in one batch."""
    import torch
    L, M = 4 * math.pi, 256
    rng = np.random.default_rng(64)
    xs = [W.cosine_positions(rng, 1 << 17, L, 0.4, 0.5), rng.normal(0.3 * L, 0.02 * L, 1 << 17) % L,
          W.cosine_positions(rng, 3000, L, 0.4, 0.5)]
    xs = [to_gpu(x) for x in xs]
    kap = W.log_kappas(1.0, 120.0, 6)
    announce("deposit moments, batch")
    bt = gpu.Batch(xs, [L] * 3, [M] * 3, kap, n_cv=4096)
    try:
        for _ in range(2):
            bt.run()
            torch.cuda.synchronize()
            for s, x in enumerate(xs):
                _, _, am = gpu.cv_scan(x[:4096], L, kap)
                ks = float(kap[int(host(am)[0])])
                assert host(bt.kappa_star)[s] == ks
                pilot = gpu.deposit(x, L, M, kappa=ks)
                assert np.array_equal(host(bt.pilot[s]), host(pilot)), s
                k_i, _, _ = gpu.adapt_widths(x, L, pilot, ks, 0.5)
                assert np.array_equal(host(bt.kappa_i[s]), host(k_i)), s
                assert np.array_equal(host(bt.rho[s]), host(gpu.deposit(x, L, M, kappa_i=k_i))), s
    finally:
        bt.close()
