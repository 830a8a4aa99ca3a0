"""The Fourier moments on both sides of their plan's lines: the direct form and
the matrix forms (particles x rounds of 1024 modes about 16384), the matrix forms'
tiles and mode blocks at counts beyond that line, and scans whose workspace
holds fewer rows than the chip takes; against the oracle's Fourier sums.

Tolerance: that of the Fourier scan, 1e-12 of each objective value and pair sum
and 1e-13 of the double sum a pair sum is the difference of."""
import math

import numpy as np
import pytest

import workloads as W
from oracle import cv as ocv
from oracle.vonmises import conv2_at_zero, kernel
from tests.gpu_util import announce, host, rel_err, to_gpu

pytestmark = pytest.mark.gpu
L = 4 * math.pi


def check(x, kap, cv, sums):
    n, B = len(x), len(kap)
    cv, sums = host(cv), host(sums)
    ref_cv, S1, S2 = ocv.cv_curve_fourier(x, L, kap)
    assert rel_err(cv, ref_cv).max() <= 1e-12
    tot1 = n * conv2_at_zero(kap, L) + 2 * S1
    tot2 = n * kernel(0.0, kap, L) + 2 * S2
    assert np.all(np.abs(sums[:B] - S1) <= 1e-12 * np.abs(S1) + 1e-13 * tot1)
    assert np.all(np.abs(sums[B:] - S2) <= 1e-12 * np.abs(S2) + 1e-13 * tot2)


@pytest.mark.parametrize("n", [16383, 16384, 16385, 16385 + 512])
@pytest.mark.parametrize("top", [0.3, 144.0, 146.0, 640.0, 2700.0, 6300.0, 11200.0, 12500.0, 13000.0])
def test_forms_and_tiles(gpu, n, top):
    x = W.cosine_positions(np.random.default_rng([91, n]), n, L, 0.4, 0.5)
    kap = np.array([0.02, 0.3, 1.0]) * top
    announce("moment plans", n, top)
    cv, sums, _ = gpu.cv_scan_fourier(to_gpu(x), L, kap)
    check(x, kap, cv, sums)


@pytest.mark.parametrize("n", [1820, 1821, 2500])
def test_many_mode_blocks(gpu, n):
    x = W.cosine_positions(np.random.default_rng([92, n]), n, L, 0.4, 0.5)
    kap = np.array([3.0, 4e4, 1e6])
    announce("moment plans, blocks", n)
    cv, sums, _ = gpu.cv_scan_fourier(to_gpu(x), L, kap)
    check(x, kap, cv, sums)


@pytest.mark.parametrize("n,top", [(17000, 100.0), (17000, 1e4), (30001, 1e4), (30001, 3e3), (18000, 2e5)])
def test_scans_of_few_concentrations(gpu, n, top):
    """Their workspace holds fewer rows; the batched engine plans alike."""
    import torch
    x = W.cosine_positions(np.random.default_rng([93, n]), n, L, 0.4, 0.5)
    for kap in (np.array([top]), np.array([0.1, 0.5, 1.0]) * top):
        announce("moment plans, few", n, top, len(kap))
        cv, sums, am = gpu.cv_scan(to_gpu(x), L, kap)
        check(x, kap, cv, sums)
        bt = gpu.Batch([to_gpu(x), to_gpu(x[:700])], [L] * 2, [64] * 2, kap)
        try:
            for _ in range(2):
                bt.run()
                torch.cuda.synchronize()
                assert torch.equal(bt.cv[0], cv)
                assert torch.equal(bt.cv[1], gpu.cv_scan(to_gpu(x[:700]), L, kap)[0])
        finally:
            bt.close()


def test_batch_without_a_place_for_the_objective(gpu):
    """Sets whose caller takes no objective, with lists that go through the
    moments, over pairs, and both."""
    import torch
    xs = [to_gpu(W.cosine_positions(np.random.default_rng([94, n]), n, L, 0.4, 0.5)) for n in (2, 40, 900)]
    for kap in (W.log_kappas(1.0, 1e5, 64), W.log_kappas(0.01, 0.04, 3)):
        rho = [torch.empty(2, dtype=torch.float64, device="cuda") for _ in xs]
        ks = torch.empty(len(xs), dtype=torch.float64, device="cuda")
        sets = [gpu.kde_batch_set(x.shape[0], x.data_ptr(), L, 2, 0, 0, None, None, r.data_ptr(), None,
                                  ks[k:].data_ptr()) for k, (x, r) in enumerate(zip(xs, rho))]
        h = gpu.kde_batch_plan(sets, gpu.KDE_F64, kap)
        try:
            need = gpu.kde_batch_workspace_size(h)
            ws = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
            at = (ws.data_ptr() + 255) // 256 * 256
            announce("moment plans, batch without objective", len(kap))
            gpu.kde_batch_run(h, at, need)
            torch.cuda.synchronize()
            for k, x in enumerate(xs):
                am = int(host(gpu.cv_scan(x, L, kap)[2])[0])
                assert host(ks)[k] == kap[am]
        finally:
            gpu.kde_batch_destroy(h)


@pytest.mark.parametrize("n,B", [(2, 8), (10, 8), (10, 9), (64, 8), (64, 9), (256, 8), (257, 8)])
def test_small_samples_whose_lists_need_the_pairs_too(gpu, n, B):
    x = W.cosine_positions(np.random.default_rng([96, n]), n, L, 0.4, 0.5)
    kap = W.log_kappas(1.0, 1e4, B)
    announce("moment plans, small lists", n, B)
    cv, sums, am = gpu.cv_scan(to_gpu(x), L, kap)
    ref, S1, S2 = ocv.cv_curve(x, L, kap)
    first = conv2_at_zero(kap, L) / n + 2 * S1 / n ** 2
    assert np.all(np.abs(host(cv) - ref) <= 1e-12 * np.maximum(np.abs(ref), 0.01 * first))
    bt = gpu.Batch([to_gpu(x)], [L], [16], kap)
    try:
        bt.run()
        assert np.array_equal(host(bt.cv[0]), host(cv))
    finally:
        bt.close()
