"""FP64 direct kernel on either side of the rule that cuts the support into
ranges (17 to 64 coordinates: one round of workgroups while a range of it holds
fewer than 128 entries): distances against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from tests._parity import dist_rel_err, oracle_state_to_gpu

pytestmark = pytest.mark.gpu


# tiles of 256 of the nb rows, 3 to 9, against the support of k + win b
# entries in 768 (33 to 64 coordinates) or 1024 workgroups
@pytest.mark.parametrize("d,k,b,win,nb", [
    (40, 3, 8192, 3, 768), (40, 3, 8192, 3, 769), (64, 3, 2048, 6, 1792), (64, 3, 2048, 6, 1793),
    (17, 3, 8192, 2, 1793), (17, 3, 8192, 2, 1792), (32, 3, 8192, 2, 2049), (33, 2, 300, 2, 300), (65, 2, 700, 2, 513),
])
def test_distances(d, k, b, win, nb):
    from paper_2410_05902_amd import Model
    rng = np.random.default_rng(d + nb)
    n = 5000
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
              precision="fp64")
    m.init_centers(init)
    m.set_state(oracle_state_to_gpu(orc.state(), init, k, win, b))
    Q = rng.integers(0, n, nb).astype(np.int32)
    D = m.assign(Q, want_D=True)["D"].cpu().numpy()
    S = np.unique(np.concatenate([rng.integers(0, nb, 30), np.arange(nb - 4, nb)]))
    ref = orc.distances(Q[S], threads=8)
    assert dist_rel_err(D[S], ref["D"], 1.0 + np.broadcast_to(ref["N"], ref["D"].shape)).max() <= 1e-9
