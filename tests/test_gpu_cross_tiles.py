"""The general MFMA cross kernel (more than 128 coordinates) on either side of
the rule that picks its batch tile, and at the tiles' edges: every distance of
sampled rows against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from tests._parity import dist_rel_err, oracle_state_to_gpu

pytestmark = pytest.mark.gpu

# relative error of a product x.y: the split's dropped terms and FP32 sums, or BF16
# factors (a kernel value's error is 2 |x| |y| / kappa times it, a distance's twice that)
REL = {"bf16x3": lambda d: 3.0 * 2.0 ** -16 + 3.0 * d * 2.0 ** -24, "bf16x1": lambda d: 2.0 ** -8 + d * 2.0 ** -24}


# 128-row tiles of the full support (a multiple of 128 rows) by 128 batch rows: 512 in
# BF16 and 2048 in FP32 take tiles of 128 batch rows, fewer take 64
@pytest.mark.parametrize("precision,k,b,win,nb", [
    ("bf16x3", 7, 1024, 8, 1024), ("bf16x3", 7, 1024, 8, 897), ("bf16x3", 7, 1024, 8, 896), ("bf16x3", 7, 1024, 8, 65),
    ("bf16x1", 7, 1024, 8, 1023), ("bf16x1", 7, 1024, 8, 129),
    ("fp32", 5, 2048, 8, 2048), ("fp32", 5, 2048, 8, 1921), ("fp32", 5, 2048, 8, 1920), ("fp32", 5, 2048, 8, 31),
])
def test_distances(precision, k, b, win, nb):
    from paper_2410_05902_amd import Model
    rng = np.random.default_rng(b + nb)
    n, d = 6000, 160
    means = rng.standard_normal((k, d))
    comp = rng.integers(0, k, n)
    X = (means[comp] + 0.5 * rng.standard_normal((n, d))).astype(np.float32)
    kappa = 4.0 * d
    init = np.array([np.flatnonzero(comp == j)[0] for j in range(k)], np.int32)
    orc = O.Oracle(X, k, win, O.GAUSS, kappa)
    orc.init_centers(init)
    for _ in range(win):
        B = rng.integers(0, n, b).astype(np.int32)
        orc.update(B, comp[B].astype(np.int32))
    m = Model(torch.from_numpy(X).cuda(), k=k, b_max=b, window=win, kernel="gauss", kernel_param=kappa,
              precision=precision, cross_impl="mfma")
    m.init_centers(init)
    m.set_state(oracle_state_to_gpu(orc.state(), init, k, win, b))
    y2 = float((X.astype(np.float64) ** 2).sum(1).max())
    tol = 1e-5 if precision == "fp32" else 1e-5 + 4.0 * REL[precision](d) * y2 / kappa
    Q = rng.integers(0, n, nb).astype(np.int32)
    D = m.assign(Q, want_D=True)["D"].cpu().numpy()
    S = np.unique(np.concatenate([rng.integers(0, nb, 40), np.arange(max(0, nb - 70), nb), np.arange(min(nb, 4))]))
    ref = orc.distances(Q[S], threads=8)
    assert dist_rel_err(D[S], ref["D"], 1.0 + np.broadcast_to(ref["N"], ref["D"].shape)).max() <= tol
