"""Self-norm blocks cut into tasks of 8 slot rows (rows of at most 8
coordinates) and of two 16-row tiles (matrix-core forms): cluster sizes around
both, and centers with no rows, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from tests.test_gpu_parity import lockstep

pytestmark = pytest.mark.gpu

COUNTS = [[1, 8, 16, 32, 0], [7, 9, 15, 17, 33], [31, 0, 48, 64, 65], [16, 33, 1, 49, 127]]


@pytest.mark.parametrize("d,kind,precision,impl", [
    (2, O.GAUSS, "fp32", "direct"), (8, O.LAPLACE, "fp32", "direct"), (7, O.GAUSS, "fp64", "direct"),
    (9, O.POLY2, "fp32", "direct"), (3, O.GAUSS, "fp32", "mfma"), (40, O.GAUSS, "fp32", "mfma"),
    (90, O.GAUSS, "fp32", "mfma"), (128, O.GAUSS, "fp32", "mfma"), (150, O.GAUSS, "fp32", "mfma"),
])
def test_lockstep(d, kind, precision, impl):
    rng = np.random.default_rng(d)
    k, n = 5, 2500
    means = 4.0 * np.eye(k, d) if d >= k else 2.0 / np.sqrt(d) * (np.arange(k) - 2.0)[:, None] * np.ones((1, d))
    comp = np.arange(n) % k
    X = (means[comp] + 0.3 * rng.standard_normal((n, d)) / np.sqrt(d)).astype(np.float32)
    param = {O.GAUSS: 8.0, O.LAPLACE: 8.0, O.POLY2: 1.0}[kind]
    rows = [np.flatnonzero(comp == j) for j in range(k)]
    batches = [np.concatenate([rng.choice(rows[j], c) for j, c in enumerate(cs) if c]).astype(np.int32)
               for cs in COUNTS]
    init = np.array([r[0] for r in rows], np.int32)
    lockstep(X, k, 3, kind, param, init, [rng.permutation(b) for b in batches], precision, impl=impl, b_max=256)


@pytest.mark.parametrize("d,kind,precision,impl", [
    (5, O.LAPLACE, "fp32", "direct"), (20, O.GAUSS, "fp64", "direct"), (40, O.GAUSS, "fp32", "mfma"),
])
@pytest.mark.parametrize("used", [[0, 499], [3, 67, 68, 132, 498], [250]])
def test_empty_centers(d, kind, precision, impl, used):
    # runs of empty centers shorter and longer than a wave between those with rows
    rng = np.random.default_rng(d + len(used))
    k, n = 500, 2000
    means = rng.standard_normal((k, d)) * 3.0
    comp = np.arange(n) % k
    X = (means[comp] + 0.1 * rng.standard_normal((n, d)) / np.sqrt(d)).astype(np.float32)
    rows = np.flatnonzero(np.isin(comp, used))
    init = np.arange(k, dtype=np.int32)
    batches = [rng.choice(rows, 150).astype(np.int32) for _ in range(4)]
    lockstep(X, k, 4, kind, 4.0 * d, init, batches, precision, impl=impl, b_max=256)


@pytest.mark.parametrize("d,kind,precision,impl", [
    (5, O.LAPLACE, "fp32", "direct"), (20, O.GAUSS, "fp64", "direct"), (40, O.GAUSS, "fp32", "mfma"),
    (150, O.GAUSS, "fp32", "mfma"),
])
@pytest.mark.parametrize("sizes", [[1023, 1024, 1024, 1000], [1023, 1025, 1100], [2047, 300], [1, 2500, 5]])
def test_large_center(d, kind, precision, impl, sizes):
    # supports of one center below, at and past 2048 entries, laid out slot by slot
    # (with its initial point while that has a weight), beside a small one
    rng = np.random.default_rng(d + sum(sizes))
    k, n = 3, 3000
    means = 3.0 * np.eye(k, d)
    comp = np.where(np.arange(n) < 60, np.arange(n) % k, 1)
    X = (means[comp] + 0.4 * rng.standard_normal((n, d)) / np.sqrt(d)).astype(np.float32)
    big, small = np.flatnonzero(comp == 1), np.flatnonzero(comp == 2)
    batches = [rng.permutation(np.concatenate([rng.choice(big, s), rng.choice(small, 3)])).astype(np.int32)
               for s in sizes]
    batches.append(batches[0][:100].copy())
    lockstep(X, k, 3, kind, 8.0, np.arange(k, dtype=np.int32), batches, precision, impl=impl, b_max=2560)
