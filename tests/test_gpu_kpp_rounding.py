"""Kernel k-means++ selection where a running sum rounds differently over rows
that weigh nothing: the pick stays beside the crossing.

The rows' D2 are exact here (the linear kernel on one coordinate, first pick
0), a handful of blocks of 256 rows hold one row of weight each, and the blocks
between them weigh 0.  A parallel prefix sum may come out larger at a block of
weight 0 than at the block before it; u puts the target between the two."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

BLOCK, LANES = 256, 64


def _scan(v):
    """The inclusive prefix sums of 64 lanes, by doubling strides."""
    v = v.copy()
    o = 1
    while o < LANES:
        t = v.copy()
        t[o:] += v[:-o]
        v, o = t, 2 * o
    return v


def _case(per):
    """X (n, 1), u_1, and the two rows beside the crossing.  per: blocks per
    thread of the selection's first level (1: the gap lies between stretches;
    more: between the blocks of a stretch)."""
    for seed in range(2000):
        rng = np.random.default_rng(seed)
        nb = 40
        w = np.zeros(nb)
        # (squares of 24-bit values are exact; their sums over several binades are not)
        w[:5] = (0.5 + rng.random(5)) * 0.5 ** rng.integers(0, 8, 5)
        w[20:23] = (0.5 + rng.random(3)) * 0.5 ** rng.integers(0, 8, 3)
        w = w.astype(np.float32)
        n = per * 1000 * BLOCK if per > 1 else nb * BLOCK
        X = np.zeros((n, 1), np.float32)
        at = (np.arange(nb) * BLOCK + 128)[w > 0]
        X[at, 0] = w[w > 0]
        b = np.zeros(LANES)
        b[:nb] = X[np.arange(nb) * BLOCK + 128, 0].astype(np.float64) ** 2
        inc = _scan(b)
        # a stretch's blocks are added one after another
        tot = sum(b.tolist()) if per > 1 else inc[-1]
        gap = np.flatnonzero(inc[5:20] > inc[4])
        if gap.size == 0 or not inc[4] < tot:
            continue
        u = inc[4] / tot
        for cand in (u, np.nextafter(u, 0), np.nextafter(u, 1)):
            if inc[4] <= cand * tot < inc[5 + gap[0]]:
                return X, float(cand), (int(at[4]), int(at[5]))
    raise AssertionError("no such case")


@pytest.mark.parametrize("per", [1, 40])
def test_pick_beside_the_crossing(per):
    from paper_2410_05902_amd import Model
    X, u, beside = _case(per)
    m = Model(torch.from_numpy(X).cuda(), k=2, b_max=64, window=2, kernel="linear")
    picks = m.init_kmeanspp(np.array([0.0, u])).cpu().numpy()
    assert picks[0] == 0 and picks[1] in beside, (picks, beside)
