"""The table update on matrix cores over every kind of segment a tile of 32
grouped entries can hold: one segment through several tiles, one end inside,
many ends, ends at the tile's and the half's edges, a support that ends inside
a tile, and centers without entries between them.  Distances of every point
after two steps against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from tests._parity import dist_rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [32, 64, 96, 128, 50])
@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("sizes", [
    [64, 32, 32],                        # ends at tile edges
    [16, 16, 16, 48],                    # ... and at the halves' edges
    [1] * 33,                            # an entry per center, past one tile
    [3, 13, 2, 14, 31, 1, 40],           # several ends, halves of both kinds
    [5, 20, 7, 20, 12, 4, 4, 4, 4, 50],  # a segment over entry 16 that ends before the first one's place
    [10, 9, 90, 1, 1, 1],                # over several tiles, then many ends
    [40, 0, 0, 21] + [0] * 70 + [30, 2],  # more centers than the window between two segments
    [200],
])
def test_segments(sizes, d, precision):
    rng = np.random.default_rng(len(sizes) * 1000 + d)
    k, n = len(sizes), 700
    # components far apart, so that the labels (and the segments) are the sizes
    means = 6.0 * rng.standard_normal((k, d))
    comp = np.concatenate([np.arange(k), rng.integers(0, k, n - k)])
    X = (means[comp] + 0.3 * rng.standard_normal((n, d))).astype(np.float32)
    kappa = 12.0 * d
    init = np.arange(k, dtype=np.int32)
    from paper_2410_05902_amd import Model
    m = Model(torch.from_numpy(X).cuda(), k=k, b_max=sum(sizes), window=0, kernel="gauss", kernel_param=kappa,
              precision=precision)
    orc = O.Oracle(X, k, 0, O.GAUSS, kappa)
    orc.init_centers(init)
    m.init_centers(init)
    everything = np.arange(n, dtype=np.int32)
    for step in range(3):
        ref = orc.distances(everything, threads=8)
        a = m.assign(everything, want_D=True)
        # FP32: the form's gate.  BF16X3: the split's relative error of a product
        # against |x||y| (3 terms of 2^-16, the FP32 sums of 3 dp terms) and the
        # norms' roundings in the exponent, twice (D holds -2 T)
        Y2 = float((X.astype(np.float64) ** 2).sum(1).max())
        rho = 3.0 * 2.0 ** -16 + 3.0 * (-(-d // 32) * 32) * 2.0 ** -24
        tol = 1e-5 if precision == "fp32" else 2.0 * (2.0 * rho * Y2 + 2.0 ** -21 * Y2) / kappa + 1e-5
        err = dist_rel_err(a["D"].cpu().numpy(), ref["D"], 1.0 + np.broadcast_to(orc.norms(), ref["D"].shape))
        assert err.max() <= tol, (step, err.max())
        if step < 2:
            B = np.concatenate([rng.choice(np.flatnonzero(comp == j), s) for j, s in enumerate(sizes)]).astype(np.int32)
            rng.shuffle(B)
            lab = m.step(B)["labels"].cpu().numpy()
            np.testing.assert_array_equal(lab, comp[B])
            orc.step(B)
