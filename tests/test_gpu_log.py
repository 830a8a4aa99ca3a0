"""The logarithm of the adaptive widths: with one particle on a node, log_geomean is
the logarithm of that node's pilot. Values whose logarithm lies within 0.02
units of half way between two doubles, random ones, and powers of two.

Tolerance: 0.52 units in the last place against long double, the bound of the
library's logarithm."""
import numpy as np
import pytest

from tests.gpu_util import announce, host, to_gpu

pytestmark = pytest.mark.gpu
HALFWAY = ["0x1.6690541228bc3p+0", "0x1.64942ec93bb2dp+0", "0x1.6940d132949efp+0", "0x1.666fba457f281p+0",
           "0x1.6e6cf106d2927p-1", "0x1.6568cfebd9665p+0", "0x1.698cc1e1d62d7p+0", "0x1.6267c6092d6dfp+0",
           "0x1.6f5ad8516aa4fp-1", "0x1.682db5beeba6bp+0", "0x1.6520259ce9e0bp+0", "0x1.6a342dc5f9d93p-1"]


def test_logarithm(gpu):
    rng = np.random.default_rng(95)
    v = np.concatenate([[float.fromhex(h) for h in HALFWAY], np.exp(rng.uniform(-0.3465, 0.3465, 200)),
                        np.exp(rng.uniform(-300.0, 300.0, 200)), 2.0 ** np.arange(-1022, 1024, 93)])
    x = to_gpu(np.zeros(1))
    announce("log", len(v))
    out = []
    for value in v:
        _, lg, floored = gpu.adapt_widths(x, 1.0, to_gpu(np.array([value, value])), 1.0, 0.5)
        out.append(float(host(lg)[0]))
    ref = np.log(v.astype(np.longdouble))
    unit = np.spacing(np.abs(ref.astype(np.float64)))
    err = np.abs(np.array(out).astype(np.longdouble) - ref) / np.where(ref == 0, 1, unit)
    assert float(err.max()) <= 0.52, v[np.argmax(err)]
