"""Re-scored rows whose candidates hold many support entries: they are listed
and finished by every workgroup of a later launch (the update where it is the
small one, a launch of its own else), or by their own workgroup when there is
no room.  Distances, labels, margins and the update's grouping against the
oracle on the same state."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from paper_2410_05902_amd import workloads as W
from tests._parity import dist_rel_err, oracle_state_to_gpu

pytestmark = pytest.mark.gpu


# rows are listed from n = 8192 on (none at 1000 and 3000); d = 160 takes the other
# cross kernel, k = 600 the general update (test_gpu_rescore_split.py: the rules' edges)
@pytest.mark.parametrize("n,d,k,b", [(1000, 64, 5, 700), (3000, 64, 5, 1000), (40000, 128, 5, 1025),
                                     (40000, 160, 4, 640), (40000, 64, 600, 900), (60000, 32, 1100, 800)])
def test_listed_rows(n, d, k, b):
    rng = np.random.default_rng(n + d + k)
    # one wide blob shared by two near-equal initial centers, the rest far off
    X = 0.3 * rng.standard_normal((n, d))
    X[: n // 50] += 4.0 * rng.standard_normal((n // 50, d))
    X = X.astype(np.float32)
    kappa = 2.0 * W.median_pairwise_distance(X, 0) ** 2
    init = rng.choice(n // 50, k, replace=False) if k < n // 50 else rng.choice(n, k, replace=False)
    init = init.astype(np.int32)
    init[0], init[1] = n - 1, n - 2
    win = 3
    from paper_2410_05902_amd import Model
    m = Model(torch.from_numpy(X).cuda(), k=k, b_max=b, window=win, kernel="gauss", kernel_param=kappa,
              precision="bf16x3", tie_delta=5e-3)
    orc = O.Oracle(X, k, win, O.GAUSS, kappa)
    orc.init_centers(init)
    m.init_centers(init)
    eN = m.selfnorm_error_bound()
    total = 0
    for i in range(1, 6):
        B = rng.integers(0, n, b).astype(np.int32)
        m.set_state(oracle_state_to_gpu(orc.state(), init, k, win, b))
        a = m.assign(B, want_D=True)
        total += m.rescore_count(reset=True)
        out = m.step(B, want_objective=True)
        ref = orc.step(B, threads=8)
        # the step scores as the assignment does
        assert torch.equal(a["labels"], out["labels"]) and torch.equal(a["mind"], out["mind"])
        sel = ref["margin"] > 2.0 * eN
        lab = a["labels"].cpu().numpy()
        np.testing.assert_array_equal(lab[sel], ref["labels"][sel])
        assert sel.mean() > 0.9
        # every row within the BF16 form's distance tolerance
        D = a["D"].cpu().numpy()
        assert dist_rel_err(D, ref["D"], 1.0 + np.broadcast_to(ref["N"], ref["D"].shape)).max() <= 1e-2
        # rows within the re-scoring threshold: FP64 values up to the self norms' error
        near = np.flatnonzero(ref["margin"] < 2e-3)
        best = ref["D"].argmin(1)
        err = np.abs(D[near, best[near]] - ref["D"][near, best[near]])
        assert err.size == 0 or err.max() <= eN + 1e-12
        # the update grouped the batch by these labels, in batch order
        st = m.get_state()
        r = (i - 1) % win
        np.testing.assert_array_equal(np.diff(st["slot_off"][r]), np.bincount(lab, minlength=k))
        np.testing.assert_array_equal(st["slot_idx"][r][:b], B[np.argsort(lab, kind="stable")])
    assert total > 20  # the data makes rows to re-score
