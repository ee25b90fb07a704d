"""Bandwidths at the ends of the working type's range and past them, in the
forms that divide by the bandwidth (the VALU Gram kernels and the FP64 cross
term): center norms, distances and labels against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from tests._parity import dist_rel_err, oracle_state_to_gpu

pytestmark = pytest.mark.gpu

INF = float("inf")
# the bar of the precision forms: 1e-5 in FP32; FP64 sums of at most 400 terms
TOL = {"fp32": 1e-5, "fp64": 1e-12}


# (width 8 ... 64: rows in registers, 70: the general Gram kernel)
@pytest.mark.parametrize("d", [2, 16, 30, 60, 70])
@pytest.mark.parametrize("kernel,precision,param,scale", [
    ("laplace", "fp32", INF, 1.0), ("laplace", "fp32", 1e39, 1.0), ("laplace", "fp32", 1e-39, 1.0),
    ("gauss", "fp32", INF, 1.0), ("gauss", "fp32", 1e-39, 1.0),
    ("laplace", "fp64", INF, 1.0), ("laplace", "fp64", 1e-310, 1.0), ("gauss", "fp64", 1e-310, 1.0),
    ("gauss", "fp64", INF, 1.0),
    # distances of the bandwidth's own size
    ("laplace", "fp32", 1e38, 1e37), ("laplace", "fp32", 1e-30, 1e-31), ("laplace", "fp32", 2.0, 0.1),
    ("laplace", "fp64", 1e38, 1e37), ("laplace", "fp64", 1e-37, 1e-38), ("gauss", "fp64", 1e-70, 1e-36),
])
def test_norms_and_distances(kernel, precision, param, scale, d):
    from paper_2410_05902_amd import Model
    rng = np.random.default_rng(d)
    n, k, b, win = 900, 4, 150, 2
    X = (scale * rng.standard_normal((n, d)) / d).astype(np.float32)
    kind = {"laplace": O.LAPLACE, "gauss": O.GAUSS}[kernel]
    orc = O.Oracle(X, k, win, kind, param)
    m = Model(torch.from_numpy(X).cuda(), k=k, b_max=b, window=win, kernel=kernel, kernel_param=param,
              precision=precision, cross_impl="direct")
    init = np.arange(k, dtype=np.int32)
    orc.init_centers(init)
    # batches of rows 4..453, each row once: equal rows at a bandwidth below
    # FP32's range have no FP32 cross term, so rows scored are in no center
    order = k + rng.permutation(3 * b).astype(np.int32)
    Q = np.arange(600, n, dtype=np.int32)
    for i in range(3):
        B = order[i * b:(i + 1) * b]
        orc.update(B, rng.integers(0, k, b))  # every center holds rows, also where all distances tie
        m.set_state(oracle_state_to_gpu(orc.state(), init, k, win, b))
        np.testing.assert_allclose(m.center_norms(), orc.norms(), rtol=TOL[precision], atol=0)
        S = Q if precision == "fp32" else np.concatenate([Q, B])
        ref = orc.distances(S)
        D = m.assign(S, want_D=True)["D"].cpu().numpy()
        assert dist_rel_err(D, ref["D"], 1.0 + np.broadcast_to(ref["N"], D.shape)).max() <= TOL[precision]
    # a step takes its Gram blocks by another plan
    m.step(Q[:b])
    assert np.isfinite(m.center_norms()).all()
