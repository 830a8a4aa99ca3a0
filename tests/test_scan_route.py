"""The concentrations that the double CV scan takes through the Fourier moments
(kappa up to (n / 3 pi)^2): their pair sums are the double sums less the
diagonal, so the rule rests on the diagonal n K(0) never exceeding a few times
S2 there, wherever the particles lie. On the CPU, the oracle's two routes
(direct pair sums, Fourier moments) at the bound, over positions that make S2
small; on the GPU, lists that straddle the bound against the direct sums, and
the same bits from the allocation-free form.

Tolerances: the double sums carry about ten rounding units (the oracle's
moments about 50: its phases are not reduced) and the diagonal is at most
twice the sum it is taken from, so 1e-13 for the oracle's routes; the scan's
own 1e-12 on the GPU."""
import math

import numpy as np
import pytest

import workloads as W
from oracle import cv as ocv
from oracle.vonmises import kernel
from tests.gpu_util import announce, host, rel_err, to_gpu


def limit(n):
    return (n / (3 * math.pi)) ** 2


def positions(kind, n, L, kappa):
    rng = np.random.default_rng([47, n])
    s = L / (2 * math.pi * math.sqrt(kappa))  # the kernel's width
    if kind == "even":
        return (np.arange(n) + 0.37) / n * L
    if kind == "jittered":
        return (np.arange(n) + 0.3 * rng.random(n)) / n * L
    if kind == "pairs":
        return np.repeat((np.arange((n + 1) // 2) + 0.2) / ((n + 1) // 2) * L, 2)[:n]
    if kind == "comb":  # as many particles as fit three widths apart, the rest on one point
        k = min(n, int(L / (3 * s)))
        return np.concatenate([(np.arange(k) * 3 * s) % L, np.full(n - k, 0.5 * L)])
    if kind == "cluster":
        return rng.normal(0.4 * L, 0.5 * s + 0.004 * L, n) % L
    return W.cosine_positions(rng, n, L, 0.5, 2 * math.pi / L)


KINDS = ["even", "jittered", "pairs", "comb", "cluster", "random"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [3, 17, 160, 700])
def test_diagonal_is_bounded_by_the_pair_sum_at_the_limit(kind, n):
    L = 4 * math.pi
    k = limit(n)
    x = positions(kind, n, L, k)
    S1, S2 = ocv.pair_sums(x, L, [k])
    assert n * float(kernel(0.0, k, L)) <= 2.6 * S2[0]
    F1, F2 = ocv.pair_sums_fourier(x, L, [k])
    assert abs(F1[0] - S1[0]) <= 1e-13 * S1[0] and abs(F2[0] - S2[0]) <= 1e-13 * S2[0]


@pytest.mark.gpu
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [3, 17, 160, 700, 1500])
def test_lists_that_straddle_the_limit(gpu, kind, n):
    L = 4 * math.pi
    k = limit(n)
    x = positions(kind, n, L, k)
    kap = np.array([0.0, 0.1 * k, 0.7 * k, k * (1 - 1e-13), k * (1 + 1e-13), 1.5 * k, 4.0 * k])
    announce("scan route", kind, n)
    cv, sums, am = (host(t) for t in gpu.cv_scan(to_gpu(x), L, kap))
    ref_cv, S1, S2 = ocv.cv_curve(x, L, kap)
    B = len(kap)
    first = (n / n ** 2) * np.array([float(kernel(0.0, q, L)) for q in kap]) + 2 * S1 / n ** 2
    assert np.all(np.abs(cv - ref_cv) <= 1e-12 * np.maximum(np.abs(ref_cv), 0.01 * first))
    skipped = math.exp(-70.0) * n * n / 2 * np.array([float(kernel(0.0, q, L)) for q in kap])
    assert np.all(np.abs(sums[:B] - S1) <= 1e-12 * S1 + skipped)
    assert np.all(np.abs(sums[B:] - S2) <= 1e-12 * S2 + skipped)
    b = ocv.cv_argmin(ref_cv)
    assert int(am[0]) == b or abs(ref_cv[int(am[0])] - ref_cv[b]) <= 2e-12 * np.abs(ref_cv).max()


@pytest.mark.gpu
@pytest.mark.parametrize("n", [2, 300, 5000])
def test_noalloc_and_null_outputs_give_the_same_bits(gpu, n):
    import torch
    L = 4 * math.pi
    x = to_gpu(W.cosine_positions(np.random.default_rng([48, n]), n, L, 0.3, 0.5))
    kap = np.array([0.0, 0.5, 20.0, 3e3, 1e5, 1e9])
    announce("scan route, noalloc", n)
    cv, sums, am = gpu.cv_scan(x, L, kap)
    dom = gpu.kde_domain(L, 2, gpu.KDE_F64, 0, 0)
    cv2 = torch.full_like(cv, -1.0)
    sums2 = torch.full_like(sums, -1.0)
    am2 = torch.full_like(am, -1)
    gpu.kde_cv_scan_noalloc(dom, n, x, kap, cv2, sums2, am2)
    assert torch.equal(cv, cv2) and torch.equal(sums, sums2) and torch.equal(am, am2)
    gpu.kde_cv_scan_noalloc(dom, n, x, kap, cv2.fill_(0.0), None, None)
    assert torch.equal(cv, cv2)


@pytest.mark.gpu
def test_non_finite_position_reaches_every_concentration(gpu):
    L = 4 * math.pi
    x = W.cosine_positions(np.random.default_rng(49), 400, L, 0.3, 0.5)
    x[123] = np.nan
    gpu.kde_numeric_check()
    announce("scan route, non-finite")
    cv, _, _ = gpu.cv_scan(to_gpu(x), L, [1.0, 1e3, 1e5])  # through the moments and over pairs
    assert np.all(np.isnan(host(cv)))
    assert gpu.kde_numeric_check() == gpu.KDE_NUMERIC_POSITION
