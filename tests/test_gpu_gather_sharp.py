"""The double gather through the modes where most concentrations of a workgroup
are too sharp for the series: its particles are summed over the nodes, two to a
thread and the remainder one; against calls too small for the modes (1e-13 of the
largest value: the same terms, in the order of more lanes).
Concentrations on both sides of the near-node and exponent-table lines."""
import math

import numpy as np
import pytest

from tests.gpu_util import announce, host, to_gpu

pytestmark = pytest.mark.gpu
L, M = 4 * math.pi, 256


@pytest.mark.parametrize("n", [131072, 300001, 262144 * 4 + 1500])
@pytest.mark.parametrize("k_lo,k_hi", [(2500.0, 9000.0), (1e4, 1e9)])
def test_every_particle_over_the_nodes(gpu, n, k_lo, k_hi):
    rng = np.random.default_rng([78, n])
    x = rng.uniform(-L, 2 * L, n)
    kap = np.exp(rng.uniform(math.log(k_lo), math.log(k_hi), n))
    kap[5::4096] = 20.0  # (too few for a workgroup to take the series)
    F = to_gpu(rng.standard_normal(M))
    announce("gather sharp", n, k_lo)
    out = host(gpu.gather(to_gpu(x), L, F, kappa_i=to_gpu(kap)))
    at = np.concatenate([rng.choice(n, 4000, replace=False), [0, 5, 4101, n - 1]])
    few = np.concatenate([host(gpu.gather(to_gpu(x[a]), L, F, kappa_i=to_gpu(kap[a]))) for a in np.array_split(at, 4)])
    # a call on few particles splits a node sum over more lanes: the same terms in another order
    assert np.all(np.abs(out[at] - few) <= 1e-13 * np.abs(few).max())
