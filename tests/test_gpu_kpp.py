"""Kernel k-means++ seeding against the oracle: every pick equal, where the
update passes rows over (clusters, near and exact copies of picks) and where
its row layout has edges (block and workgroup sizes, 4-byte rows, tails)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O

pytestmark = pytest.mark.gpu

KNAME = {O.GAUSS: "gauss", O.LAPLACE: "laplace", O.LINEAR: "linear", O.POLY2: "poly2"}


def _picks(X, kind, param, k, u, ld):
    from paper_2410_05902_amd import Model
    n, d = X.shape
    buf = torch.full((n, ld), float("nan"), device="cuda")  # columns past d are never read
    buf[:, :d] = torch.from_numpy(X)
    m = Model(buf[:, :d], k=k, b_max=64, window=2, kernel=KNAME[kind], kernel_param=param)
    return m.init_kmeanspp(u).cpu().numpy()


@pytest.mark.parametrize("n,d,pad,kind", [
    (255, 2, 0, O.GAUSS), (256, 7, 0, O.GAUSS), (257, 8, 0, O.LAPLACE), (1025, 32, 0, O.LAPLACE),
    (5000, 33, 0, O.GAUSS), (5000, 35, 1, O.GAUSS), (3001, 130, 2, O.GAUSS), (3001, 64, 0, O.LAPLACE),
    ((1 << 19) + 77, 5, 3, O.GAUSS), ((1 << 19) + 77, 3, 0, O.LAPLACE),
    (2000, 6, 0, O.LINEAR), (2000, 6, 0, O.POLY2),
])
def test_picks_equal_the_oracles(n, d, pad, kind):
    rng = np.random.default_rng(n + d)
    c, k = 12, 40 if n < 100000 else 14
    means = 4.0 * rng.standard_normal((c, d))
    X = (means[rng.integers(0, c, n)] + 0.3 * rng.standard_normal((n, d))).astype(np.float32)
    X[n // 2:n // 2 + 40] = X[0]                          # exact copies
    X[n // 3:n // 3 + 40] = X[1] * np.float32(1 + 1e-6)   # near copies
    param = {O.GAUSS: 2.0 * d, O.LAPLACE: 2.0 * d}.get(kind, 1.0)
    u = rng.random(k)
    np.testing.assert_array_equal(_picks(X, kind, param, k, u, d + pad), O.kmeanspp(X, kind, param, k, u))


@pytest.mark.parametrize("kind,param", [(O.GAUSS, 1e-3), (O.GAUSS, 1e9), (O.LAPLACE, 1e-2), (O.LAPLACE, 1e9)])
def test_picks_at_the_bandwidths_ends(kind, param):
    """Kernel values that are all 0 or within rounding of 1."""
    rng = np.random.default_rng(5)
    X = rng.standard_normal((4000, 9)).astype(np.float32)
    u = rng.random(30)
    np.testing.assert_array_equal(_picks(X, kind, param, 30, u, 9), O.kmeanspp(X, kind, param, 30, u))


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_picks_with_rows_that_are_not_finite(bad):
    rng = np.random.default_rng(6)
    X = rng.standard_normal((1500, 8)).astype(np.float32)
    X[700, 3] = bad
    u = rng.random(10)
    from paper_2410_05902_amd import Model
    m = Model(torch.from_numpy(X).cuda(), k=10, b_max=64, window=2, kernel="gauss", kernel_param=8.0, validate=False)
    np.testing.assert_array_equal(m.init_kmeanspp(u).cpu().numpy(), O.kmeanspp(X, O.GAUSS, 8.0, 10, u))


def test_identical_rows():
    X = np.ones((600, 4), np.float32)
    u = np.random.default_rng(7).random(5)
    np.testing.assert_array_equal(_picks(X, O.GAUSS, 1.0, 5, u, 4), O.kmeanspp(X, O.GAUSS, 1.0, 5, u))
