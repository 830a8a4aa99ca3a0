"""The float deposit by node pairs, on both sides of its lines (65,536
particles; even grids of 32 to 256 nodes), against the double deposit of the
same positions and widths, and the batched engine with the same bits.

Tolerance: the float deposit's 1e-6 of a node (its terms' error; the density
here has no empty stretch, so no node is small)."""
import math

import numpy as np
import pytest

import workloads as W
from tests.gpu_util import announce, host, rel_err, to_gpu

pytestmark = pytest.mark.gpu
L = 4 * math.pi


@pytest.mark.parametrize("n", [65535, 65536, 131587])
@pytest.mark.parametrize("M", [30, 31, 32, 34, 62, 66, 100, 128, 254, 255, 256, 258])
def test_against_double(gpu, n, M):
    rng = np.random.default_rng([101, n, M])
    x = W.cosine_positions(rng, n, L, 0.4, 0.5).astype(np.float32)
    kap = (10.0 ** rng.uniform(-1, 2, n)).astype(np.float32)
    announce("deposit pairs", n, M)
    got = host(gpu.deposit(to_gpu(x), L, M, kappa_i=to_gpu(kap)))
    ref = host(gpu.deposit(to_gpu(x.astype(np.float64)), L, M, kappa_i=to_gpu(kap.astype(np.float64))))
    assert rel_err(got, ref).max() <= 1e-6
    got = host(gpu.deposit(to_gpu(x), L, M, kappa=20.0))
    ref = host(gpu.deposit(to_gpu(x.astype(np.float64)), L, M, kappa=20.0))
    assert rel_err(got, ref).max() <= 1e-6


def test_non_finite_position(gpu):
    n, M = 70001, 100
    x = W.cosine_positions(np.random.default_rng(102), n, L, 0.4, 0.5).astype(np.float32)
    x[[3, 69999]] = [np.nan, np.inf]
    gpu.kde_numeric_check()
    announce("deposit pairs, non-finite")
    assert np.all(np.isnan(host(gpu.deposit(to_gpu(x), L, M, kappa=20.0))))
    assert gpu.kde_numeric_check() == gpu.KDE_NUMERIC_POSITION


def test_batch_gives_the_same_bits(gpu):
    rng = np.random.default_rng(103)
    sizes, grids = [70001, 3000, 90000], [100, 128, 31]
    xs = [to_gpu(W.cosine_positions(rng, n, L, 0.4, 0.5).astype(np.float32)) for n in sizes]
    kap = W.log_kappas(1.0, 120.0, 5)
    announce("deposit pairs, batch")
    bt = gpu.Batch(xs, [L] * 3, grids, kap, n_cv=2048)
    try:
        bt.run()
        for s, (x, M) in enumerate(zip(xs, grids)):
            ks = float(host(bt.kappa_star)[s])
            assert np.array_equal(host(bt.pilot[s]), host(gpu.deposit(x, L, M, kappa=ks))), s
            assert np.array_equal(host(bt.rho[s]), host(gpu.deposit(x, L, M, kappa_i=bt.kappa_i[s]))), s
    finally:
        bt.close()
