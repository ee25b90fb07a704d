"""Small supports of the direct kernel: ranges of at least 8 entries, summed in
FP64, and the scoring's batched reads of the partials, over batch sizes
around the ranges' and rows' edges, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from tests.test_gpu_parity import lockstep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,k,b,win,kind,precision", [
    (2, 3, 256, 4, O.GAUSS, "fp32"), (2, 1, 7, 1, O.GAUSS, "fp32"), (5, 2, 257, 3, O.LAPLACE, "fp32"),
    (9, 4, 513, 2, O.POLY2, "fp64"), (33, 2, 300, 4, O.LAPLACE, "fp32"), (70, 3, 90, 4, O.GAUSS, "fp64"),
    (3, 2, 1024, 12, O.GAUSS, "fp32"),
])
def test_lockstep(d, k, b, win, kind, precision):
    rng = np.random.default_rng(d * 1000 + b)
    n = 3000
    means = 3.0 * rng.standard_normal((k, d))
    comp = rng.integers(0, k, n)
    X = (means[comp] + 0.5 * rng.standard_normal((n, d))).astype(np.float32)
    param = {O.GAUSS: 2.0 * d, O.LAPLACE: 2.0 * d, O.POLY2: 1.0}[kind]
    init = np.array([np.flatnonzero(comp == j)[0] for j in range(k)], np.int32)
    batches = [rng.integers(0, n, b).astype(np.int32) for _ in range(win + 2)]
    lockstep(X, k, win, kind, param, init, batches, precision, impl="direct", b_max=b)
