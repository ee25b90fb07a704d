"""Timed cases of mini-batch kernel k-means, each through the package's public
entry points (Model, batch_objective).

A case is one of six programs:

- "fit":   the early-stopping loop of Algorithm 2 (Model.fit) on small data;
- "steps": a run of Algorithm 2 from given initial centers, a few iterations
           past a full window, the labels and distances of every batch kept;
- "seed":  kernel k-means++ seeding, the start of every run;
- "label": every row of the data assigned to trained centers and the labels
           scored against reference labels (the end of every run);
- "table": Algorithm 1 without truncation, on the table of cross terms;
- "grad":  one gradient step's work when tuning the bandwidth: forward and
           backward of the batch objective.

The listed sizes are those of the repository's workloads; draw() spreads the
same programs over the ranges around them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2410_05902_amd import Model, workloads
from paper_2410_05902_amd.autograd import batch_objective

DEV = "cuda"


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest program: 2-D blobs, where launches and host work count;
        # checked calls (the default), early stopping on
        dict(name="fit_blobs2d_fp32", kind="fit", data="blobs", n=2000, d=2, k=3, b=256, window=4, kernel="gauss",
             precision="fp32", lr="beta", tau=0, steps=4, validate=True),
        # the benchmark workload: a large Gaussian mixture in the BF16 split form
        dict(name="steps_gmm128_bf16x3", kind="steps", data="gmm", n=1_000_000, d=128, k=100, b=4096, window=4,
             kernel="gauss", precision="bf16x3", lr="beta", tau=0, steps=10, validate=False),
        # a mid-size mixture in plain FP32, calls checked as by default
        dict(name="steps_gmm64_fp32", kind="steps", data="gmm", n=100_000, d=64, k=50, b=2048, window=4,
             kernel="gauss", precision="fp32", lr="beta", tau=0, steps=10, validate=True),
        # image-like rows: many coordinates, few centers, a longer window
        dict(name="steps_proto784_fp32", kind="steps", data="proto", n=70_000, d=784, k=10, b=1024, window=8,
             kernel="gauss", precision="fp32", lr="beta", tau=0, steps=12, validate=False),
        # the Laplacian kernel: many centers, the largest batch
        dict(name="steps_l1mix32_fp32", kind="steps", data="l1mix", n=4_000_000, d=32, k=1000, b=8192, window=4,
             kernel="laplace", precision="fp32", lr="beta", tau=0, steps=8, validate=False),
        # the FP64 form, a reference run beside the others
        dict(name="steps_gmm64_fp64", kind="steps", data="gmm", n=100_000, d=64, k=50, b=1024, window=4,
             kernel="gauss", precision="fp64", lr="beta", tau=0, steps=8, validate=True),
        # seeding of the benchmark workload and of the Laplacian one
        dict(name="seed_gmm128", kind="seed", data="gmm", n=1_000_000, d=128, k=100, b=4096, window=4,
             kernel="gauss", precision="bf16x3", lr="beta", tau=0, steps=0, validate=False),
        dict(name="seed_l1mix32", kind="seed", data="l1mix", n=4_000_000, d=32, k=1000, b=8192, window=4,
             kernel="laplace", precision="fp32", lr="beta", tau=0, steps=0, validate=False),
        # the last call of a run: a label for every row, scored
        dict(name="label_gmm128_bf16x3", kind="label", data="gmm", n=1_000_000, d=128, k=100, b=4096, window=4,
             kernel="gauss", precision="bf16x3", lr="beta", tau=0, steps=6, validate=True),
        # the untruncated form: Gaussian on the matrix cores, Laplacian on the
        # vector units (a 16 GB table, the largest case)
        dict(name="table_gmm128_bf16x3", kind="table", data="gmm", n=1_000_000, d=128, k=100, b=4096, window=0,
             kernel="gauss", precision="bf16x3", lr="beta", tau=0, steps=3, validate=False),
        dict(name="table_l1mix32_fp32", kind="table", data="l1mix", n=4_000_000, d=32, k=1000, b=8192, window=0,
             kernel="laplace", precision="fp32", lr="beta", tau=0, steps=2, validate=False),
        # bandwidth tuning: forward and backward of the differentiation form
        dict(name="grad_gmm64_fp32", kind="grad", data="gmm", n=100_000, d=64, k=50, b=2048, window=4,
             kernel="gauss", precision="fp32", lr="beta", tau=0, steps=6, validate=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fit", "steps", "steps", "steps", "seed", "label", "table", "grad"])
    c = dict(kind=kind, data="gmm", n=_log(rng, 5000, 400_000), d=_log(rng, 16, 200), k=_log(rng, 3, 300),
             b=_log(rng, 100, 4096), window=rng.choice([2, 3, 4, 4, 4, 6, 8]), kernel="gauss",
             precision=rng.choice(["fp32", "bf16x3"]), lr="beta", tau=0, steps=6, validate=rng.random() < 0.5)
    if kind == "fit":
        c.update(data="blobs", n=_log(rng, 1000, 20_000), d=rng.randint(2, 8), k=rng.randint(2, 8),
                 b=_log(rng, 64, 512), precision="fp32", steps=4, validate=True)
    elif kind == "steps":
        which = rng.choice(["gauss", "gauss", "laplace", "proto", "fp64"])
        if which == "laplace":
            c.update(data="l1mix", d=_log(rng, 4, 64), k=_log(rng, 10, 1000), b=_log(rng, 200, 8192),
                     kernel="laplace", precision="fp32")
        elif which == "proto":
            c.update(data="proto", n=_log(rng, 5000, 70_000), d=_log(rng, 200, 784), k=rng.randint(5, 20),
                     b=_log(rng, 100, 2048), precision="fp32")
        elif which == "fp64":
            c.update(precision="fp64", b=_log(rng, 100, 1024), d=_log(rng, 8, 100), window=4)
        else:
            c.update(tau=rng.choice([0, 0, 200]))
        c["steps"] = min(10, c["window"] + 3)
    elif kind == "seed":
        c.update(n=_log(rng, 5000, 1_000_000), k=_log(rng, 5, 100), precision="fp32", steps=0, validate=False)
        if rng.random() < 0.4:
            c.update(data="l1mix", kernel="laplace", d=_log(rng, 8, 64))
    elif kind == "label":
        c.update(n=_log(rng, 20_000, 300_000), validate=True)
    elif kind == "table":
        c.update(d=_log(rng, 16, 128), k=_log(rng, 5, 100), window=0, steps=3)
        if rng.random() < 0.4:
            c.update(data="l1mix", kernel="laplace", precision="fp32", d=_log(rng, 8, 64))
    elif kind == "grad":
        c.update(validate=True, k=_log(rng, 5, 100), n=_log(rng, 5000, 100_000))
    c["k"] = min(c["k"], c["n"] // 20)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _data(case, seed):
    """Rows of a mixture (float32, on the GPU) and the component of each."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    n, d, data = case["n"], case["d"], case["data"]
    c = case["k"]
    comp = torch.randint(0, c, (n,), generator=g, device=DEV, dtype=torch.int32)

    def randn(*s):
        return torch.randn(*s, generator=g, device=DEV)

    def rand(*s):
        return torch.rand(*s, generator=g, device=DEV)

    if data == "blobs":      # isotropic blobs, means U[-5, 5]^d, std 1
        means, std = 10.0 * rand(c, d) - 5.0, 1.0
    elif data == "gmm":      # Gaussian components, means N(0, I), std 0.3
        means, std = randn(c, d), 0.3
    elif data == "l1mix":    # means U[-10, 10]^d, std 0.4
        means, std = 20.0 * rand(c, d) - 10.0, 0.4
    else:                    # sparse prototypes, rows clipped to [0, 1]
        means, std = rand(c, d) * (rand(c, d) < 0.2), 0.1
    X = torch.empty(n, d, device=DEV)
    for r in range(0, n, 1 << 20):
        s = slice(r, min(n, r + (1 << 20)))
        X[s] = means[comp[s].long()] + std * randn(s.stop - s.start, d)
    if data == "proto":
        X.clamp_(0.0, 1.0)
    return X, comp


def _bandwidth(case, X):
    """(kernel parameter, sigma): sigma 1 for the blobs and 4 for the Laplacian,
    the median of the pairwise distances of 1000 rows else."""
    if case["kernel"] == "laplace":
        return 4.0, 4.0
    s = 1.0 if case["data"] == "blobs" else workloads.median_pairwise_distance(X[:1000].cpu().numpy(), 0)
    return 2.0 * s * s, s


def _inputs(case, seed):
    X, comp = _data(case, seed)
    g = torch.Generator(device=DEV).manual_seed(seed + 1)
    param, sigma = _bandwidth(case, X)
    # batches are drawn with repetition (Algorithm 1), staged on the GPU
    batches = torch.randint(0, case["n"], (max(1, case["steps"]), case["b"]), generator=g, device=DEV,
                            dtype=torch.int32)
    u = np.random.default_rng(seed).random(case["k"])
    return X, comp, param, sigma, batches, u


def _random_rows(case, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randperm(case["n"], generator=g)[:case["k"]].to(torch.int32)


def _plain_init(case):
    """Random rows as initial centers where k is large (k-means++ else)."""
    return case["kernel"] == "laplace"


def prepare(case, seed):
    X, comp, param, sigma, batches, u = _inputs(case, seed)
    m = Model(X, k=case["k"], b_max=case["b"], window=case["window"], kernel=case["kernel"], kernel_param=param,
              precision=case["precision"], lr=case["lr"], tau=case["tau"], validate=case["validate"])
    s = dict(kind=case["kind"], model=m, batches=[batches[i] for i in range(case["steps"])], u=u, k=case["k"])
    if case["kind"] != "seed":
        s["init"] = _random_rows(case, seed).to(DEV) if _plain_init(case) else m.init_kmeanspp(u)
    if case["kind"] in ("label", "grad"):  # trained centers, the window full
        m.init_centers(s["init"])
        for bt in s["batches"]:
            m.step_noout(bt)
    if case["kind"] == "label":
        s["all"] = torch.arange(case["n"], dtype=torch.int32, device=DEV)
        s["truth"] = comp
    if case["kind"] == "grad":
        s["xb"] = X[:case["b"]].clone().requires_grad_(True)
        s["sigma"] = torch.tensor(0.9 * sigma, dtype=torch.float32, requires_grad=True)
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    m, kind = s["model"], s["kind"]
    if kind == "seed":
        return m.init_kmeanspp(s["u"])
    if kind == "fit":
        m.init_centers(s["init"])
        taken, gains = m.fit(s["batches"], eps=-1.0)  # gains lie in [-1, 1]: every step runs
        return dict(taken=taken, gains=gains)
    if kind in ("steps", "table"):
        m.init_centers(s["init"])
        outs = [m.step(bt) for bt in s["batches"]]
        return dict(labels=[o["labels"] for o in outs], mind=[o["mind"] for o in outs])
    if kind == "label":
        o = m.assign(s["all"])
        ari, nmi, table = m.agreement(o["labels"], s["truth"], s["k"])
        return dict(labels=o["labels"], mind=o["mind"], margin=o["margin"], ari=ari, nmi=nmi, table=table)
    s["xb"].grad = s["sigma"].grad = None
    loss = batch_objective(m, s["xb"], s["sigma"])
    loss.backward()
    return dict(loss=float(loss), dX=s["xb"].grad, dsigma=s["sigma"].grad)


def work(case):
    """One pass: each kernel value's 2 d operations once (products counted
    once whatever the form), each input read and each output written once."""
    n, d, k, b, W, T = case["n"], case["d"], case["k"], case["b"], case["window"], case["steps"]
    kind = case["kind"]
    if kind == "seed":
        return {"bytes": 4 * n * d + 4 * k, "flops": 2 * n * d * (k - 1)}
    if kind == "table":
        return {"bytes": 4 * n * d + 8 * T * n * k + T * b * 8, "flops": 2 * d * n * (T * b + k)}
    if kind == "label":
        M = min(T, W) * b
        return {"bytes": 4 * n * d + 16 * n, "flops": 2 * d * n * M}
    if kind == "grad":
        M = min(T, W) * b
        # cross term, self norms within the centers, and the gradient of each
        # row against its own center (about 1 / k of the support)
        return {"bytes": 4 * d * (2 * b + M), "flops": 2 * d * (b * M + M * M // k + 2 * b * M // k)}
    f = by = 0
    for i in range(T):
        M = min(i, W) * b + (k if i <= W else 0)
        f += 2 * d * (b * M + b * M // k) * (2 if kind == "fit" else 1)
        by += 4 * d * b + 8 * b
    return {"bytes": by, "flops": f}


# ---------------------------------------------------------------------------
# the same in 64 bits, plain torch
# ---------------------------------------------------------------------------
def _kernel(case, A, B, param):
    """K of the rows of A (p x d) with those of B (q x d), float64."""
    if case["kernel"] == "gauss":
        D = (A * A).sum(1)[:, None] + (B * B).sum(1)[None, :]
        D.addmm_(A, B.t(), alpha=-2.0).clamp_(min=0.0)
    else:
        D = torch.zeros(A.shape[0], B.shape[0], dtype=torch.float64, device=A.device)
        At, Bt = A.t().contiguous(), B.t().contiguous()
        for t in range(A.shape[1]):
            D += (At[t][:, None] - Bt[t][None, :]).abs_()
    return D.div_(-param).exp_()


def _kpp(case, X, param, u):
    """Kernel k-means++: pick r is the first row whose running sum of
    2 - 2 max_c K(x, c) exceeds u_r times the whole sum."""
    n = X.shape[0]
    picks = [min(n - 1, int(math.floor(u[0] * n)))]
    D2 = torch.full((n,), math.inf, dtype=torch.float64, device=X.device)
    X64 = X.double()
    for r in range(1, len(u)):
        c = X64[picks[-1]]
        for q in range(0, n, 1 << 18):
            diff = X64[q:q + (1 << 18)] - c
            e = (diff * diff).sum(1) if case["kernel"] == "gauss" else diff.abs().sum(1)
            D2[q:q + (1 << 18)] = torch.minimum(D2[q:q + (1 << 18)], 2.0 - 2.0 * torch.exp(-e / param))
        cs = torch.cumsum(D2, 0)
        picks.append(int(torch.searchsorted(cs, cs[-1:] * float(u[r]), right=True).clamp(max=n - 1)))
    return torch.tensor(picks, dtype=torch.long, device=X.device)


class _Exact:
    """Algorithm 2 (window > 0) or 1 (window 0) with every center as a list of
    weighted points, all in float64."""

    def __init__(self, case, X, param, init):
        self.c, self.X, self.param, self.k = case, X, param, case["k"]
        self.W = case["window"] if case["window"] > 0 else 1 << 30
        self.init = init.long()
        self.i = 1
        self.cinit = torch.ones(self.k, dtype=torch.float64, device=X.device)
        self.bat = []  # [rows, labels, per-center coefficient, counts]

    def support(self):
        rows, lab, w = [], [], []
        if bool((self.cinit != 0).any()):
            rows.append(self.init)
            lab.append(torch.arange(self.k, device=self.X.device))
            w.append(self.cinit)
        for r, l, cf, _ in self.bat:
            rows.append(r)
            lab.append(l)
            w.append(cf[l])
        rows, lab, w = torch.cat(rows), torch.cat(lab), torch.cat(w)
        keep = w != 0
        return self.X[rows[keep]].double(), lab[keep], w[keep]

    def cross(self, A, Y, lab, w, param):
        """sum over the entries of each center of w K(a, y): (p x k)."""
        order = torch.argsort(lab, stable=True)
        Y, lab, w = Y[order], lab[order], w[order]
        hot = torch.zeros(Y.shape[0], self.k, dtype=torch.float64, device=A.device)
        hot[torch.arange(Y.shape[0], device=A.device), lab] = w
        out = torch.empty(A.shape[0], self.k, dtype=torch.float64, device=A.device)
        step = max(1, (1 << 27) // max(1, Y.shape[0]))
        for q in range(0, A.shape[0], step):
            out[q:q + step] = _kernel(self.c, A[q:q + step], Y, param) @ hot
        return out

    def norms(self, Y, lab, w, param):
        N = torch.zeros(self.k, dtype=torch.float64, device=Y.device)
        for j in torch.unique(lab).tolist():
            s = lab == j
            Yj, wj = Y[s], w[s]
            step = max(1, (1 << 27) // max(1, Yj.shape[0]))
            for q in range(0, Yj.shape[0], step):
                N[j] += wj[q:q + step] @ (_kernel(self.c, Yj[q:q + step], Yj, param) @ wj)
        return N

    def distances(self, A, param=None):
        param = self.param if param is None else param
        Y, lab, w = self.support()
        N = self.norms(Y, lab, w, param)
        return 1.0 - 2.0 * self.cross(A, Y, lab, w, param) + N[None, :]

    def step(self, batch):
        rows = batch.long()
        mind, lab = self.distances(self.X[rows].double()).min(1)
        cnt = torch.bincount(lab, minlength=self.k).double()
        a = torch.sqrt(cnt / rows.numel())
        self.cinit *= 1.0 - a
        for bt in self.bat:
            bt[2] = bt[2] * (1.0 - a)
        self.bat.append([rows, lab, torch.where(cnt > 0, a / cnt.clamp(min=1.0), torch.zeros_like(a)), cnt])
        if len(self.bat) > self.W:
            self.bat.pop(0)
        if self.i > self.W:
            self.cinit.zero_()
        tau = self.c["tau"]
        if tau > 0:  # keep the newest batches up to the one at which the counts reach tau
            seen = torch.zeros(self.k, dtype=torch.float64, device=self.X.device)
            drop = torch.zeros(self.k, dtype=torch.bool, device=self.X.device)
            first = self.i + 1 - len(self.bat)
            for q in range(len(self.bat) - 1, -1, -1):
                self.bat[q][2] = torch.where(drop, torch.zeros_like(seen), self.bat[q][2])
                seen = seen + self.bat[q][3]
                if first + q > 1:
                    drop = drop | (seen >= tau)
            self.cinit = torch.where(drop, torch.zeros_like(seen), self.cinit)
        self.i += 1
        return mind


def exact(case, seed):
    if case["kind"] == "seed":
        return None  # row numbers only
    X, comp, param, sigma, batches, u = _inputs(case, seed)
    init = _random_rows(case, seed).to(DEV) if _plain_init(case) else _kpp(case, X, param, u)
    E = _Exact(case, X, param, init)
    kind = case["kind"]
    if kind == "fit":
        gains = []
        for bt in batches:
            f = float(E.step(bt).mean())
            gains.append(f - float(E.distances(X[bt.long()].double()).min(1)[0].mean()))
        return dict(taken=None, gains=gains)
    minds = [E.step(bt) for bt in batches]
    if kind in ("steps", "table"):
        return dict(labels=None, mind=minds)
    if kind == "label":
        mind = torch.empty(case["n"], dtype=torch.float64, device=DEV)
        margin = torch.empty_like(mind)
        Y, lab, w = E.support()
        N = E.norms(Y, lab, w, param)
        for q in range(0, case["n"], 1 << 14):
            D = 1.0 - 2.0 * E.cross(X[q:q + (1 << 14)].double(), Y, lab, w, param) + N[None, :]
            two = D.topk(min(2, case["k"]), dim=1, largest=False)[0]
            mind[q:q + (1 << 14)] = two[:, 0]
            margin[q:q + (1 << 14)] = two[:, -1] - two[:, 0]
        return dict(labels=None, mind=mind, margin=margin, ari=None, nmi=None, table=None)
    # the differentiation form, support points and weights held constant
    sg = torch.tensor(float(torch.tensor(0.9 * sigma, dtype=torch.float32)), dtype=torch.float64, device=DEV)
    kappa = float(2.0 * sg * sg)
    xb = X[:case["b"]].double()
    D = E.distances(xb, kappa)
    mind, best = D.min(1)
    Y, lab, w = E.support()
    dX = torch.zeros_like(xb)
    ds = 0.0
    for j in torch.unique(best).tolist():
        r, s = best == j, lab == j
        Yj, wj, xj = Y[s], w[s], xb[r]
        Kx = _kernel(case, xj, Yj, kappa)
        dX[r] = 2.0 / (case["b"] * float(sg) ** 2) * ((Kx @ wj)[:, None] * xj - (Kx * wj) @ Yj)
        d2 = -kappa * torch.log(Kx.clamp(min=1e-300))
        dn = 0.0
        step = max(1, (1 << 27) // max(1, Yj.shape[0]))
        for q in range(0, Yj.shape[0], step):
            Kn = _kernel(case, Yj[q:q + step], Yj, kappa)
            dn += float(wj[q:q + step] @ ((Kn * (-kappa * torch.log(Kn.clamp(min=1e-300)))) @ wj))
        ds += float(-2.0 * (Kx * d2 * wj).sum() + int(r.sum()) * dn) / float(sg) ** 3
    return dict(loss=float(mind.mean()), dX=dX, dsigma=torch.tensor(ds / case["b"], dtype=torch.float64))
