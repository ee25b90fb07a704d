"""Rows re-scored in FP64 on either side of the rules that list and split them:
n below and at the least that lists rows, few listed rows (each split over
workgroups) and many (none split), more candidates or centers than a split
takes.  Listed rows are finished by k_rescore or by the small update; here every
row is re-scored, so that every distance to a candidate is FP64 up to the self
norms' error, and all of them hold more entries than a scoring workgroup takes."""
import os
import re

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from tests._parity import oracle_state_to_gpu

pytestmark = pytest.mark.gpu

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_05902_amd", "csrc")


def _constant(name, text):
    return int(re.search(r"constexpr int %s = (\d+);" % name, text).group(1))


# rows: listed at once; parts of a row: the most (up to 16) that the 256 workgroups have for each
@pytest.mark.parametrize("n,d,k,win,rows,listed,parts", [
    # no room for the list's scratch: the scoring workgroups do all, a few rows one after
    # another, many a wave to each (here from 7 rows on at 64 coordinates, from 58 at 160)
    (8191, 64, 3, 2, 40, False, 0), (8191, 64, 3, 2, 4, False, 0), (8191, 160, 3, 2, 64, False, 0),
    (8191, 64, 600, 2, 70, False, 0),
    (8192, 64, 3, 2, 1, True, 16), (8192, 64, 3, 2, 16, True, 16), (8192, 64, 3, 2, 17, True, 8),
    (8192, 64, 3, 2, 128, True, 2), (8192, 64, 3, 2, 129, True, 1), (9000, 128, 16, 2, 1000, True, 1),
    (9000, 128, 17, 2, 30, False, 0),     # more candidates than a split takes
    (9000, 160, 3, 2, 20, True, 8), (9000, 160, 3, 2, 300, True, 1),  # the general cross kernel's partials
    (9000, 64, 3, 8, 20, True, 8), (9000, 64, 3, 8, 300, True, 1),    # the general update
    (9000, 64, 600, 2, 20, True, 1),     # more centers than k_rescore's threads
])
def test_rescored_rows(n, d, k, win, rows, listed, parts):
    from paper_2410_05902_amd import Model
    rng = np.random.default_rng(n + d + k + rows)
    head = open(os.path.join(SRC, "rescore.h")).read()
    near = min(k, 17) if k < 600 else 3
    # one blob for the centers 0 .. near - 1, the others' single points far off
    X = (0.3 * rng.standard_normal((n, d))).astype(np.float32)
    if k > near:
        X[near:k] += (2.0 * rng.standard_normal((k - near, d))).astype(np.float32)
    kappa = 2.0 * d * 0.09
    b = 1500
    orc = O.Oracle(X, k, win, O.GAUSS, kappa)
    init = np.arange(k, dtype=np.int32)
    orc.init_centers(init)
    for _ in range(2):
        B = rng.integers(k, n, b).astype(np.int32)
        orc.update(B, rng.integers(0, near, b))
    # by construction: every row's candidates are the `near` centers, 3000 entries
    assert (2 * b > _constant("kRescoreOwnEntries", head)) and "R.split = L.n >= 8192;" in open(
        os.path.join(SRC, "kernels_score.hip")).read()
    assert listed == (n >= 8192 and near <= _constant("kRescoreMaxCand", head))
    if listed:
        most = 1
        while most < _constant("kRescoreMaxParts", head) and rows * 2 * most <= _constant("kRescoreWGs", head):
            most *= 2
        assert parts == (most if k <= _constant("kRescoreThreads", head) else 1)

    m = Model(torch.from_numpy(X).cuda(), k=k, b_max=b, window=win, kernel="gauss", kernel_param=kappa,
              precision="bf16x3", tie_delta=0.5)
    m.init_centers(init)
    state = oracle_state_to_gpu(orc.state(), init, k, win, b)
    m.set_state(state)
    eN = m.selfnorm_error_bound()
    Q = rng.integers(k, n, rows).astype(np.int32)
    ref = orc.distances(Q)
    D = ref["D"]
    assert (D[:, :near].max(1) < D.min(1) + 0.4).all() and (k == near or (D[:, near:].min(1) > D.min(1) + 0.6).all())

    def check(out):
        lab, mind = out["labels"].cpu().numpy(), out["mind"].cpu().numpy()
        sel = ref["margin"] > 2.0 * eN
        np.testing.assert_array_equal(lab[sel], ref["labels"][sel])
        assert np.abs(mind - ref["mind"]).max() <= eN + 2.0 ** -23
        return lab

    m.rescore_count(reset=True)
    for _ in range(2):  # the second launch finds the list empty again
        a = m.assign(Q, want_D=True)
        check(a)
        assert np.abs(a["D"].cpu().numpy()[:, :near] - D[:, :near]).max() <= eN + 1e-12
        assert np.abs(a["margin"].cpu().numpy() - ref["margin"]).max() <= 2.0 * eN + 2.0 ** -23
        assert m.rescore_count(reset=True) == rows
    # the objective sums the re-scored rows' distances, in one chunk and over several
    for R in (Q, np.resize(Q, 2 * b + 17)):
        mind = m.assign(R)["mind"].double()
        assert m.rescore_count(reset=True) == R.size
        assert abs(m.objective(R) - float(mind.mean())) <= 1e-14
        assert m.rescore_count(reset=True) == R.size
    out = m.step(Q, want_objective=True)
    lab = check(out)
    assert m.rescore_count(reset=True) == rows
    assert abs(out["fbefore"] - ref["mind"].mean()) <= eN + 2.0 ** -23
    st = m.get_state()
    r = 2 % win  # batch 3
    np.testing.assert_array_equal(np.diff(st["slot_off"][r]), np.bincount(lab, minlength=k))
    np.testing.assert_array_equal(st["slot_idx"][r][:rows], Q[np.argsort(lab, kind="stable")])
