"""Workspace sizes are part of what a caller plans with: whatever route a call
takes, a scan asks for the pair layout's arrays (the histogram of the cell sort,
the packed particles, the slots' sums, their column sums and the raw sums), the
Fourier scans for the budget of their longest series, a batch for its sets' arrays.
kde_cv_scan_noalloc takes every scan whose pair layout fits its array."""
import ctypes
import math

import numpy as np
import pytest

import paper_1804_11174_amd as kde


def dom(prec, shape=0):
    return kde.kde_domain(4 * math.pi, 64, prec, shape, 0)


def ceil_div(a, b):
    return -(-a // b)


def carve(*arrays):
    used = 0
    for size in arrays:
        used = ceil_div(used, 256) * 256 + size
    return used


def pair_layout(n, B, prec):
    cells = min(max(n // 32, 1), 8192)
    blocks = min(max(ceil_div(n, 2048), 1), 128)
    tiles = ceil_div(n, 256)
    slots = min(tiles * (tiles + 1) // 2, 32768)
    packed = 24 if prec == kde.KDE_F64 else 4
    return carve(4 * cells * blocks, packed * n, 16 * B * slots, 16 * B * ceil_div(slots, 128) + 8, 16 * B)


@pytest.mark.parametrize("prec", [kde.KDE_F64, kde.KDE_F32])
@pytest.mark.parametrize("shape", [kde.KDE_SHAPE_VONMISES, kde.KDE_SHAPE_TRIANGLE])
def test_scans_ask_for_the_pair_layout(prec, shape):
    ns = list(range(2, 700)) + [int(2 ** (k / 7)) + d for k in range(66, 210) for d in (-1, 0, 1)]
    for n in ns:
        for B in (1, 2, 8, 32, 64):
            assert kde.kde_workspace_size(kde.KDE_OP_CV_SCAN, dom(prec, shape), n, B) == pair_layout(n, B, prec), (n, B)


@pytest.mark.parametrize("B,n", [(1, 851776), (8, 697664), (16, 521536), (32, 220191), (64, 54528)])
def test_noalloc_limits_in_double(B, n):
    room = 24 << 20
    assert kde.kde_workspace_size(kde.KDE_OP_CV_SCAN, dom(kde.KDE_F64), n, B) <= room
    assert kde.kde_workspace_size(kde.KDE_OP_CV_SCAN, dom(kde.KDE_F64), n + 1, B) > room


@pytest.mark.parametrize("op,n,B,most", [
    (kde.KDE_OP_CV_FOURIER, 2, 1, 511632), (kde.KDE_OP_CV_FOURIER, 1000, 32, 2769920),
    (kde.KDE_OP_CV_FOURIER, 4096, 1, 658576), (kde.KDE_OP_CV_FOURIER, 20011, 32, 3944448),
    (kde.KDE_OP_CV_FOURIER, 65536, 1, 5062800), (kde.KDE_OP_CV_FOURIER, 1 << 20, 32, 12019200),
    (kde.KDE_OP_ADAPT_EXACT, 2, 0, 658448), (kde.KDE_OP_ADAPT_EXACT, 4096, 0, 837904),
    (kde.KDE_OP_ADAPT_EXACT, 65536, 0, 5737488), (kde.KDE_OP_ADAPT_EXACT, 1 << 20, 0, 18361872)])
def test_fourier_scans_keep_their_budget(op, n, B, most):
    for prec in (kde.KDE_F64, kde.KDE_F32):
        assert kde.kde_workspace_size(op, dom(prec), n, B) <= most


@pytest.mark.parametrize("prec,sets,B,most", [
    (kde.KDE_F64, [(3000, 64, 0)], 16, 119560), (kde.KDE_F32, [(3000, 64, 0)], 16, 59400),
    (kde.KDE_F64, [(30000, 256, 0), (1000, 64, 0), (7, 2, 0)], 64, 9044488),
    (kde.KDE_F32, [(30000, 256, 0), (1000, 64, 0), (7, 2, 0)], 64, 8424456),
    (kde.KDE_F64, [(200000, 256, 65536)], 8, 10288904), (kde.KDE_F32, [(200000, 256, 65536)], 8, 8978184)])
def test_batches_keep_their_sizes(prec, sets, B, most):
    somewhere = 256  # a plan only keeps the addresses
    arr = [kde.kde_batch_set(n, somewhere, 12.5, M, 0, n_cv, somewhere, somewhere, somewhere, somewhere, somewhere)
           for n, M, n_cv in sets]
    h = kde.kde_batch_plan(arr, prec, np.geomspace(1.0, 1e4, B))
    try:
        assert kde.kde_batch_workspace_size(h) <= most
    finally:
        kde.kde_batch_destroy(h)
