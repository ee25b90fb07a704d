"""The table update on matrix cores at every padded row width (32, 64, 96, 128
coordinates): every coordinate of the batch entries is staged."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from tests._parity import dist_rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [17, 33, 65, 80, 96, 97, 128])
@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
def test_widths(d, precision):
    rng = np.random.default_rng(d)
    k, n, b = 5, 900, 150
    means = 2.0 * rng.standard_normal((k, d))
    comp = np.concatenate([np.arange(k), rng.integers(0, k, n - k)])
    X = (means[comp] + 0.3 * rng.standard_normal((n, d))).astype(np.float32)
    kappa = 4.0 * d
    from paper_2410_05902_amd import Model
    m = Model(torch.from_numpy(X).cuda(), k=k, b_max=b, window=0, kernel="gauss", kernel_param=kappa,
              precision=precision)
    orc = O.Oracle(X, k, 0, O.GAUSS, kappa)
    init = np.arange(k, dtype=np.int32)
    orc.init_centers(init)
    m.init_centers(init)
    # BF16X3: relative error of the split product (3 terms of 2^-16, FP32 sums of
    # 3 dp terms) and the norms' roundings in the exponent, twice (D holds -2 T)
    Y2 = float((X.astype(np.float64) ** 2).sum(1).max())
    rho = 3.0 * 2.0 ** -16 + 3.0 * (-(-d // 32) * 32) * 2.0 ** -24
    tol = 1e-5 if precision == "fp32" else 2.0 * (2.0 * rho * Y2 + 2.0 ** -21 * Y2) / kappa + 1e-5
    everything = np.arange(n, dtype=np.int32)
    for step in range(2):
        ref = orc.distances(everything, threads=8)
        D = m.assign(everything, want_D=True)["D"].cpu().numpy()
        want = ref["D"]
        err = dist_rel_err(D, want, 1.0 + np.broadcast_to(orc.norms(), want.shape))
        assert err.max() <= tol, (step, err.max(), tol)
        if step == 0:
            B = rng.integers(0, n, b).astype(np.int32)
            m.step(B)
            orc.step(B)
