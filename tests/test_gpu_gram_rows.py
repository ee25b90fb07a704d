"""Self-norm blocks on matrix cores in tasks of one and of two row tiles: batches
on either side of the rule between them in one run, with clusters of 0 to some
hundred rows (tiles part-filled, one and two), against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from tests.test_gpu_parity import lockstep

pytestmark = pytest.mark.gpu


# k (W + 1) tasks per row tile and 64 column rows: 640 at 64 rows per center, 1600 at 65
@pytest.mark.parametrize("d,precision", [(32, "fp32"), (60, "bf16x3"), (96, "fp32"), (128, "fp32")])
def test_lockstep(d, precision):
    rng = np.random.default_rng(d)
    k, n, win = 40, 6000, 3
    means = 3.0 * rng.standard_normal((k, d)) / np.sqrt(d) * 2.0
    comp = np.arange(n) % k
    X = (means[comp] + 0.3 * rng.standard_normal((n, d)) / np.sqrt(d)).astype(np.float32)
    rows = [np.flatnonzero(comp == j) for j in range(k)]
    few = [0, 1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65]

    def batch(b):
        c = np.array([few[j % len(few)] for j in rng.permutation(k)])
        c[-1] += b - c.sum()  # the rest in one center
        assert c[-1] > 0
        return rng.permutation(np.concatenate([rng.choice(rows[j], m) for j, m in enumerate(c) if m])).astype(np.int32)

    batches = [batch(b) for b in (2560, 2561, 2600, 1600, 2560)]
    init = np.array([r[0] for r in rows], np.int32)
    lockstep(X, k, win, O.GAUSS, 8.0, init, batches, precision, impl="mfma", b_max=2600)
