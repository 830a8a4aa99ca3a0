"""The column sums' two ways (one launch up to 4096 rows of 512 columns, else
two) give the same bits: the batched engine sums by rows of 128 and then
over those, so its outputs are compared with the single calls' on both sides
of the lines (the widths' rows are 256 particles, the deposits' a chunk)."""
import math

import numpy as np
import pytest

import workloads as W
from tests.gpu_util import announce, host, to_gpu

pytestmark = pytest.mark.gpu
L = 4 * math.pi


@pytest.mark.parametrize("n,M", [(32768, 64), (32769, 513), (70001, 512), (1048576, 40), (1048577, 33), (2097153, 16)])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_batch_gives_the_same_bits(gpu, n, M, dtype):
    rng = np.random.default_rng([111, n])
    x = to_gpu(W.cosine_positions(rng, n, L, 0.4, 0.5).astype(dtype))
    announce("column sums", n, M, dtype)
    bt = gpu.Batch([x], [L], [M], W.log_kappas(1.0, 120.0, 5), n_cv=2048)
    try:
        bt.run()
        ks = float(host(bt.kappa_star)[0])
        pilot = gpu.deposit(x, L, M, kappa=ks)
        assert np.array_equal(host(bt.pilot[0]), host(pilot))
        k_i, _, _ = gpu.adapt_widths(x, L, pilot, ks, 0.5)
        assert np.array_equal(host(bt.kappa_i[0]), host(k_i))
        assert np.array_equal(host(bt.rho[0]), host(gpu.deposit(x, L, M, kappa_i=k_i)))
    finally:
        bt.close()
