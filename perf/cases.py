"""The work that is timed: solves, unrolled learning steps and loss heads.

listed() are the cases, draw(rng) gives more of the same ranges, prepare() the
inputs (and the handle that a program keeps), run() one pass through the
public entry points, work() what a pass cannot do without, and exact() the
same outputs from plain torch in 64 bits.

Kinds, sizes from the repository's workloads and tests:
  heads      cost model, regret and weight gradient of a routing learner
  surrogate  SPO+ and perturbed Fenchel-Young losses of the same learner
  lp         create + solve one sparse LP (a program that gets a new LP)
  resolve    solve a large sparse LP, or a dense one, on a kept handle
  dense      create + solve one dense LP
  qp         create + solve one convex QP (Q low rank, CSR or dense)
  grid       create + solve a batch of min-cost flows sharing one grid
  ragged     create + solve a batch of uneven LPs
  learn      one training step through unrolled iterations of a grid batch
  portfolio  batched portfolio QPs: solve, then a gradient through T iterations

Solves run to the relative KKT tolerance 1e-4 or to a limit of iterations
where the tolerance takes longer than a pass should.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2412_09734_amd import heads
from paper_2412_09734_amd.solver import BatchSolver, Solver

DEV = "cuda"
F64 = torch.float64
EPS = 1e-4
CHECK = 64        # the default check cadence


def listed():
    return [
        # the smallest calls: a learner that trains on a few 32 x 32 grids at a time
        {"name": "heads_small", "kind": "heads", "B": 8, "n": 3968, "p": 5},
        # surrogate losses over a whole training batch, four perturbations each
        {"name": "surrogate_256", "kind": "surrogate", "B": 256, "n": 3968, "M": 4},
        # the small planted LP, new each time: latency and launches count
        {"name": "lp_small", "kind": "lp", "m": 200, "n": 400, "mean": 4.0, "family": "planted", "limit": 100000},
        # an ordinary sparse LP of odd size with skewed column lengths
        {"name": "lp_medium", "kind": "lp", "m": 30001, "n": 60013, "mean": 10.0, "family": "zipf", "limit": 2048},
        # the headline LP, a stretch of iterations on a kept handle
        {"name": "lp_large", "kind": "resolve", "m": 1000000, "n": 2000000, "mean": 10.0, "family": "zipf",
         "limit": 512},
        # a dense LP of ordinary, ragged size
        {"name": "dense_medium", "kind": "dense", "m": 1537, "n": 3001, "limit": 1024},
        # the large dense LP (6.4 GB) on a kept handle
        {"name": "dense_large", "kind": "resolve", "m": 20000, "n": 40000, "mean": 0.0, "family": "dense",
         "limit": 96},
        # one convex QP with a factor-model objective
        {"name": "qp_lowrank", "kind": "qp", "m": 2000, "n": 5000, "mean": 4.0, "q": "lowrank", "rank": 20,
         "limit": 1024},
        # the batched headline: 2,048 flows on one 32 x 32 grid
        {"name": "grid_2048", "kind": "grid", "B": 2048, "rows": 32, "cols": 32},
        # 1,024 LPs of uneven size, m from 50 to 500
        {"name": "ragged_1024", "kind": "ragged", "B": 1024, "lo": 50, "hi": 500, "density": 0.05},
        # the learning step: 256 grids through 1,000 iterations and back
        {"name": "learn_256", "kind": "learn", "B": 256, "rows": 32, "cols": 32, "p": 5, "T": 1000},
        # 512 portfolio QPs, solved and differentiated
        {"name": "portfolio_512", "kind": "portfolio", "B": 512, "n": 500, "rank": 20, "T": 1000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["heads", "surrogate", "lp", "lp", "resolve", "dense", "qp", "qp", "grid", "ragged", "learn",
                       "portfolio"])
    c = {"kind": kind}
    if kind == "heads":
        c.update(B=_log_int(rng, 1, 512), n=_log_int(rng, 24, 6000), p=rng.randint(1, 64))
    elif kind == "surrogate":
        c.update(B=_log_int(rng, 1, 256), n=_log_int(rng, 24, 6000), M=rng.randint(1, 4))
    elif kind == "lp":
        m = _log_int(rng, 40, 60000)
        c.update(m=m, n=int(m * rng.uniform(1.2, 3.0)), mean=rng.uniform(2.0, 10.0),
                 family=rng.choice(["planted", "zipf"]), limit=2048)
    elif kind == "resolve":
        c["family"] = rng.choice(["zipf", "dense"])
        if c["family"] == "zipf":
            m = _log_int(rng, 80000, 900000)
            c.update(m=m, n=int(m * rng.uniform(1.2, 2.1)), mean=10.0, limit=256)
        else:
            m = _log_int(rng, 300, 12000)
            c.update(m=m, n=min(100003, _log_int(rng, 4000, 60000000) // m + 64), mean=0.0, limit=256)
    elif kind == "dense":
        m = _log_int(rng, 20, 2500)
        c.update(m=m, n=int(m * rng.uniform(1.2, 3.0)), limit=1024)
    elif kind == "qp":
        n = _log_int(rng, 60, 6000)
        c.update(n=n, m=max(1, int(n * rng.uniform(0.05, 0.5))), mean=rng.uniform(2.0, 6.0),
                 q=rng.choice(["lowrank", "csr", "dense"]), rank=rng.randint(1, 32), limit=512)
    elif kind == "grid":
        c.update(B=_log_int(rng, 16, 1024), rows=rng.randint(6, 32), cols=rng.randint(6, 32))
    elif kind == "ragged":
        lo = rng.randint(20, 100)
        c.update(B=_log_int(rng, 16, 768), lo=lo, hi=rng.randint(lo + 1, 480), density=0.05)
    elif kind == "learn":
        c.update(B=_log_int(rng, 8, 256), rows=rng.randint(6, 32), cols=rng.randint(6, 32), p=rng.randint(2, 16),
                 T=rng.randint(100, 1000))
    else:
        c.update(B=_log_int(rng, 16, 512), n=_log_int(rng, 40, 700), rank=rng.randint(1, 32),
                 T=rng.randint(100, 900))
    return c


# ---------------------------------------------------------------------------
# inputs


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=F64)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=F64)


class Csr:
    """A sparse matrix from its sorted keys row * n + column, and its transpose."""

    def __init__(self, m, n, key, val):
        self.m, self.n, self.val = m, n, val
        self.row, self.col = key // n, key % n
        self.rowptr = self._ptr(self.row, m)
        self.perm = torch.argsort(self.col * m + self.row)
        self.colptr = self._ptr(self.col, n)

    @staticmethod
    def _ptr(idx, length):
        p = torch.zeros(length + 1, dtype=torch.int64, device=DEV)
        torch.cumsum(torch.bincount(idx, minlength=length), 0, out=p[1:])
        return p

    def operators(self, val=None):
        """(A, A') as torch CSR matrices."""
        v = self.val if val is None else val
        a = torch.sparse_csr_tensor(self.rowptr, self.col, v, (self.m, self.n))
        at = torch.sparse_csr_tensor(self.colptr, self.row[self.perm], v[self.perm], (self.n, self.m))
        return a, at

    def arrays(self):
        return dict(rowptr=self.rowptr.int(), colidx=self.col.int(), val=self.val)


def _plant(g, mul, tmul, m, n, rho=0.5, eq_frac=0.6):
    """Planted optimum for x >= 0: c, lc, uc with a known primal-dual pair."""
    supp = _rand(g, n) < rho
    x = torch.where(supp, _rand(g, n), 0.0)
    eq = _rand(g, m) < eq_frac
    y = torch.where(eq, _randn(g, m), 0.0)
    ax, slack, le = mul(x), _rand(g, m), _rand(g, m) < 0.5
    inf = torch.full((m,), math.inf, dtype=F64, device=DEV)
    lc = torch.where(eq, ax, torch.where(le, -inf, ax - slack))
    uc = torch.where(eq, ax, torch.where(le, ax + slack, inf))
    c = tmul(y) + torch.where(supp, 0.0, _rand(g, n))
    return c, lc, uc


def _pattern(g, sizes, density):
    """Keys of block-diagonal Bernoulli(density) patterns of blocks m x n."""
    n_all = sum(n for _, n in sizes)
    cells = torch.tensor([m * n for m, n in sizes], device=DEV)
    hit = torch.nonzero(torch.rand(int(cells.sum()), generator=g, device=DEV) < density).squeeze(1)
    ends = torch.cumsum(cells, 0)
    b = torch.searchsorted(ends, hit, right=True)
    local = hit - (ends - cells)[b]
    ms = torch.tensor([m for m, _ in sizes], device=DEV)
    ns = torch.tensor([n for _, n in sizes], device=DEV)
    r0, c0 = torch.cumsum(ms, 0) - ms, torch.cumsum(ns, 0) - ns
    return (r0[b] + local // ns[b]) * n_all + c0[b] + local % ns[b]


def _sparse(g, case):
    """A sparse LP: uniform rows per column, column counts Poisson-like
    ('planted') or from a power law with rows of uneven scale ('zipf')."""
    m, n, mean = case["m"], case["n"], case["mean"]
    zipf = case.get("family") == "zipf"
    if zipf:
        k = torch.arange(1, 2001, device=DEV, dtype=F64) ** -1.7948
        deg = torch.searchsorted(torch.cumsum(k / k.sum(), 0), _rand(g, n)) + 1
        deg = torch.clamp(deg, max=min(2000, m))
    else:
        deg = torch.clamp(torch.poisson(torch.full((n,), mean, dtype=F64, device=DEV), generator=g).long(), max=m)
    cols = torch.repeat_interleave(torch.arange(n, device=DEV), deg)
    rows = torch.randint(m, (cols.numel(),), generator=g, device=DEV)
    key = torch.unique(rows * n + cols)
    val = _randn(g, key.numel())
    if zipf:
        val = val * (10.0 ** (4.0 * _rand(g, m) - 2.0))[key // n]
    a = Csr(m, n, key, val)
    A, At = a.operators()
    c, lc, uc = _plant(g, lambda x: A @ x, lambda y: At @ y, m, n)
    uv = torch.full((n,), math.inf, dtype=F64, device=DEV)
    if zipf:
        uv[_rand(g, n) < 0.5] = 10.0
    return a, dict(c=c, lc=lc, uc=uc, lv=torch.zeros(n, dtype=F64, device=DEV), uv=uv)


def _dense(g, case):
    """Dense rows; few long rows are the knapsack shape, else all equalities."""
    m, n = case["m"], case["n"]
    lv, inf = torch.zeros(n, dtype=F64, device=DEV), math.inf
    if n > 40 * m:
        a = _rand(g, m, n)
        c, uc = -_rand(g, n), 0.25 * a.sum(1)
        return a, dict(c=c, lc=torch.full_like(uc, -inf), uc=uc, lv=lv, uv=torch.ones_like(lv))
    a = _randn(g, m, n)
    c, lc, uc = _plant(g, lambda x: a @ x, lambda y: y @ a, m, n, rho=0.3, eq_frac=2.0)
    return a, dict(c=c, lc=lc, uc=uc, lv=lv, uv=torch.full_like(lv, inf))


def _grid(g, case):
    """Node-arc incidence of a directed 4-neighbour grid and B flows on it."""
    r, c, B = case["rows"], case["cols"], case["B"]
    v = np.arange(r * c).reshape(r, c)
    pairs = [(v[:-1], v[1:]), (v[1:], v[:-1]), (v[:, :-1], v[:, 1:]), (v[:, 1:], v[:, :-1])]
    arcs = np.concatenate([np.stack([t.ravel(), h.ravel()], 1) for t, h in pairs])
    arcs = torch.from_numpy(arcs[np.lexsort((arcs[:, 1], arcs[:, 0]))]).to(DEV)
    m, n = r * c, arcs.shape[0]
    at = torch.arange(n, device=DEV)
    key, order = torch.sort(torch.cat([arcs[:, 0] * n + at, arcs[:, 1] * n + at]))
    one = torch.ones(n, dtype=F64, device=DEV)
    a = Csr(m, n, key, torch.cat([one, -one])[order])
    b = torch.zeros(B, m, dtype=F64, device=DEV)
    src = torch.randint(m, (B,), generator=g, device=DEV)
    snk = (src + torch.randint(1, m, (B,), generator=g, device=DEV)) % m
    k = torch.randint(1, 6, (B,), generator=g, device=DEV).double()
    rows = torch.arange(B, device=DEV)
    b[rows, src] = k
    b[rows, snk] = -k
    return a, dict(c=1.0 + 9.0 * _rand(g, B, n), lc=b, uc=b.clone(), lv=torch.zeros(B, n, dtype=F64, device=DEV),
                   uv=5.0 + 15.0 * _rand(g, B, n))


def _routing(g, B, n, p):
    """Features, true weights' costs in [1, 10] and the learner's weights."""
    f, w = _randn(g, B, n, p), _randn(g, p)
    return f, 1.0 + 9.0 * torch.sigmoid(f @ w), 0.1 * _randn(g, p)


def _ragged(g, case):
    # the sizes belong to the case, the problems to the seed
    ms = np.random.default_rng(case["B"] + case["hi"]).integers(case["lo"], case["hi"] + 1, case["B"]).tolist()
    sizes = [(m, 2 * m) for m in ms]
    m, n = sum(ms), 2 * sum(ms)
    key = _pattern(g, sizes, case["density"])
    a = Csr(m, n, key, _randn(g, key.numel()))
    A, At = a.operators()
    c, lc, uc = _plant(g, lambda x: A @ x, lambda y: At @ y, m, n)
    lv = torch.zeros(n, dtype=F64, device=DEV)
    off = np.concatenate([[0], np.cumsum(ms)])
    return a, dict(c=c, lc=lc, uc=uc, lv=lv, uv=torch.full_like(lv, math.inf)), off


def _portfolio(g, case):
    B, n = case["B"], case["n"]
    a = Csr(1, n, torch.arange(n, device=DEV), torch.ones(n, dtype=F64, device=DEV))
    one = torch.ones(B, 1, dtype=F64, device=DEV)
    v = dict(c=0.05 * _randn(g, B, n), lc=one, uc=one.clone(), lv=torch.zeros(B, n, dtype=F64, device=DEV),
             uv=torch.full((B, n), max(0.1, 4.0 / n), dtype=F64, device=DEV))
    return a, v, 0.1 * _randn(g, n, case["rank"]), 0.01 + 0.09 * _rand(g, B, n)


def _qp(g, case):
    """A planted sparse constraint set with x <= 10 and a convex Q."""
    a, v = _sparse(g, dict(case, family="planted"))
    n, r = case["n"], case["rank"]
    v["uv"] = torch.full_like(v["uv"], 10.0)
    if case["q"] == "lowrank":
        return a, v, dict(q_format="lowrank", q_factor=0.1 * _randn(g, n, r), q_diag=0.01 + 0.09 * _rand(g, n))
    if case["q"] == "dense":
        f = _randn(g, n, r) * (0.3 / math.sqrt(r))
        q = f @ f.T
        q.diagonal().add_(0.05)
        return a, v, dict(q_format="dense", q_dense=q)
    # CSR: a banded, diagonally dominant coupling of neighbours
    off = -0.2 * _rand(g, n - 1)
    i = torch.arange(n, device=DEV)
    diag = 0.5 + _rand(g, n)
    key, order = torch.sort(torch.cat([i * n + i, i[1:] * n + i[:-1], i[:-1] * n + i[1:]]))
    q = Csr(n, n, key, torch.cat([diag, off, off])[order])
    return a, v, dict(q_format="csr", q_rowptr=q.rowptr.int(), q_colidx=q.col.int(), q_val=q.val)


def _inputs(case, seed):
    """What the case is made of, from the seed: a dict of tensors."""
    g, kind = _gen(seed), case["kind"]
    if kind == "heads":
        f, ct, w = _routing(g, case["B"], case["n"], case["p"])
        return dict(f=f, ct=ct, W=w, x=_rand(g, *ct.shape), vs=_rand(g, case["B"]), gc=_randn(g, *ct.shape))
    if kind == "surrogate":
        B, n, M = case["B"], case["n"], case["M"]
        d = {k: 1.0 + 9.0 * _rand(g, B, n) for k in ("ch", "ct")}
        d.update({k: (_rand(g, B, n) < 0.02).double() for k in ("ws", "wt")})
        d.update(zs=(d["ct"] * d["ws"]).sum(1), Z=_randn(g, B, M, n), wm=(_rand(g, B, M, n) < 0.02).double())
        return d
    if kind in ("lp", "resolve") and case["family"] != "dense":
        a, v = _sparse(g, case)
        return dict(a=a, v=v)
    if kind in ("dense", "resolve"):
        a, v = _dense(g, case)
        return dict(dense=a, v=v)
    if kind == "qp":
        a, v, q = _qp(g, case)
        return dict(a=a, v=v, q=q)
    if kind == "grid":
        a, v = _grid(g, case)
        return dict(a=a, v=v)
    if kind == "ragged":
        a, v, off = _ragged(g, case)
        return dict(a=a, v=v, off=off)
    if kind == "learn":
        a, v = _grid(g, case)
        f, ct, w = _routing(g, case["B"], a.n, case["p"])
        v["c"] = ct
        return dict(a=a, v=v, f=f, W=w, vs=_rand(g, case["B"]))
    a, v, F, d = _portfolio(g, case)
    return dict(a=a, v=v, F=F, d=d)


# ---------------------------------------------------------------------------
# one pass


def _solver(case, d):
    opts = dict(eps=EPS, iteration_limit=case["limit"])
    if "dense" in d:
        return Solver(case["m"], case["n"], None, None, None, a_dense=d["dense"], **d["v"], **opts)
    return Solver(case["m"], case["n"], **d["a"].arrays(), **d["v"], **d.get("q", {}), **opts)


def _batch(case, d):
    a = d["a"]
    kw = dict(shared_a=True, batch=case["B"], m=a.m, n=a.n, **a.arrays(), **d["v"])
    if "off" in d:
        kw.update(shared_a=False, row_off=d["off"], col_off=2 * d["off"])
    if "F" in d:
        kw.update(q_factor=d["F"], q_diag=d["d"])
    return BatchSolver(**kw)


def prepare(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "resolve":
        return dict(kind=kind, handle=_solver(case, d))
    if kind in ("learn", "portfolio"):
        d["handle"] = _batch(case, d)
    return dict(d, kind=kind, case=case)


def run(s):
    kind = s["kind"]
    if kind == "heads":
        c = heads.linear_costs(s["f"], s["W"])
        loss = heads.regret(s["ct"], s["x"], s["vs"])
        return dict(c=c, loss=loss, gW=heads.linear_costs_backward(s["f"], s["gc"]))
    if kind == "surrogate":
        c = heads.spo_plus_costs(s["ch"], s["ct"])
        loss, grad = heads.spo_plus(s["ch"], s["ct"], s["ws"], s["zs"], s["wt"])
        cp = heads.pfy_costs(s["ch"], s["Z"], 0.5)
        ploss, pgrad = heads.pfy(s["ch"], s["ws"], s["Z"], 0.5, s["wm"])
        return dict(c=c, loss=loss, grad=grad, cp=cp, ploss=ploss, pgrad=pgrad)
    if kind == "resolve":
        x, y, info = s["handle"].solve()
        return dict(x=x, y=y, iterations=info["iterations"])
    if kind in ("lp", "dense", "qp"):
        with _solver(s["case"], s) as h:
            x, y, info = h.solve()
        return dict(x=x, y=y, iterations=info["iterations"])
    if kind in ("grid", "ragged"):
        with _batch(s["case"], s) as h:
            x, y, _ = h.solve()
        return dict(x=x, y=y)
    h, T = s["handle"], s["case"]["T"]
    if kind == "learn":
        ct = s["v"]["c"]
        h.update_data(c=heads.linear_costs(s["f"], s["W"]))
        x, y = h.unrolled(T)
        loss = heads.regret(ct, x, s["vs"])
        gc = h.backward(ct)[0]
        return dict(x=x, y=y, loss=loss, gc=gc, gW=heads.linear_costs_backward(s["f"], gc))
    xs, ys, _ = h.solve()
    x, _ = h.unrolled(T)
    value, gx = heads.qp_value(s["F"], s["d"], s["v"]["c"], x)
    gc, _, _, gd = h.backward(x)
    return dict(xs=xs, ys=ys, x=x, value=value, gx=gx, gc=gc, gd=gd)


# ---------------------------------------------------------------------------
# what a pass cannot do without


def work(case):
    """Inputs read once and outputs written once; a matrix too large to stay
    on the chip (256 MB) is read in each product of each iteration."""
    kind = case["kind"]
    if kind == "heads":
        N = case["B"] * case["n"]
        return {"bytes": 8 * N * (case["p"] + 4), "flops": 4 * N * case["p"] + 2 * N}
    if kind == "surrogate":
        N = case["B"] * case["n"]
        return {"bytes": 8 * N * (7 + 3 * case["M"]), "flops": N * (8 + 6 * case["M"])}
    if kind in ("lp", "resolve", "dense", "qp"):
        m, n = case["m"], case["n"]
        it = min(case["limit"], 1024)       # a typical count where the tolerance ends the solve
        dense = kind == "dense" or case.get("family") == "dense"
        nnz = m * n if dense else int(n * (10.0 if case.get("family") == "zipf" else case["mean"]))
        mat = (8 if dense else 12) * nnz
        q = 0
        if kind == "qp":
            q = {"lowrank": n * (2 * case["rank"] + 1), "csr": 3 * n, "dense": n * n}[case["q"]]
        per = 2 * mat + 8 * (8 * n + 6 * m)
        total = per * it if mat > 256e6 else mat + 8 * (q + 4 * n + 3 * m)
        return {"bytes": total, "flops": it * (4 * nnz + 2 * q + 10 * n + 10 * m)}
    if kind in ("grid", "learn"):
        r, c, B = case["rows"], case["cols"], case["B"]
        m, n = r * c, 4 * r * c - 2 * (r + c)
        it = 2 * case["T"] if kind == "learn" else 2500
        extra = (2 * case["p"] + 2) * n if kind == "learn" else 0
        return {"bytes": 8 * B * (4 * n + 3 * m + extra), "flops": B * it * (8 * n + 10 * n + 10 * m)}
    if kind == "ragged":
        m = (case["lo"] + case["hi"]) // 2
        nnz = int(case["density"] * 2 * (case["lo"] ** 2 + case["lo"] * case["hi"] + case["hi"] ** 2) / 3)
        B = case["B"]
        return {"bytes": B * (12 * nnz + 8 * (8 * m + 3 * m)), "flops": B * 1500 * (4 * nnz + 30 * m)}
    B, n, r = case["B"], case["n"], case["rank"]
    return {"bytes": 8 * B * n * 9 + 8 * n * r, "flops": B * (3 * case["T"] + 400) * n * (4 * r + 14)}


# ---------------------------------------------------------------------------
# the same outputs in 64 bits, from plain torch


class _Mul(torch.autograd.Function):
    @staticmethod
    def forward(ctx, v, fwd, bwd):
        ctx.bwd = bwd
        return fwd(v)

    @staticmethod
    def backward(ctx, g):
        return ctx.bwd(g), None, None


def _splitmix(j):
    """U(0, 1) from the counters j (SplitMix64, wrapping 64-bit arithmetic)."""
    def signed(v):
        return v - (1 << 64) if v >= 1 << 63 else v

    def shift(z, k):
        return (z >> k) & ((1 << (64 - k)) - 1)
    z = j + signed(0x9E3779B97F4A7C15)
    z = (z ^ shift(z, 30)) * signed(0xBF58476D1CE4E5B9)
    z = (z ^ shift(z, 27)) * signed(0x94D049BB133111EB)
    return shift(z ^ shift(z, 31), 11).double() * 2.0 ** -53


class Reference:
    """The restarted methods for B independent problems side by side: flat
    vectors, per-problem scalars, sums by problem. rows / cols: lengths."""

    def __init__(self, d, case):
        v = {k: t.reshape(-1) for k, t in d["v"].items()}
        self.v, B = v, case.get("B", 1)
        self.B = B
        if "dense" in d:
            a = d["dense"].clone()
            self.rows, self.cols = [a.shape[0]], [a.shape[1]]
            dr, dc = self._scale_dense(a)
            self.mul, self.tmul = (lambda x: a @ x), (lambda y: y @ a)
        else:
            a = d["a"]
            dr, dc, val = self._scale(a)
            A, At = a.operators(val)
            if "off" in d:
                off = np.diff(d["off"])
                self.rows, self.cols = off.tolist(), (2 * off).tolist()
                self.mul, self.tmul = (lambda x: A @ x), (lambda y: At @ y)
            elif B > 1:
                self.rows, self.cols = [a.m] * B, [a.n] * B
                self.mul = lambda x: (A @ x.reshape(B, -1).T.contiguous()).T.reshape(-1)
                self.tmul = lambda y: (At @ y.reshape(B, -1).T.contiguous()).T.reshape(-1)
                dr, dc = dr.repeat(B), dc.repeat(B)
            else:
                self.rows, self.cols = [a.m], [a.n]
                self.mul, self.tmul = (lambda x: A @ x), (lambda y: At @ y)
        self.lens = {n: torch.tensor(l, device=DEV) for n, l in (("r", self.rows), ("c", self.cols))}
        self.dr, self.dc = dr, dc
        self.c, self.lv, self.uv = v["c"] * dc, v["lv"] / dc, v["uv"] / dc
        self.lc, self.uc = v["lc"] * dr, v["uc"] * dr
        self.eta = 0.998 / self._norm()
        big = [torch.where(torch.isfinite(t), t.abs(), 0.0) for t in (v["lc"], v["uc"])]
        big = torch.maximum(*big)
        self.bnorm, self.cnorm = self.sum("r", big * big).sqrt(), self.sum("c", v["c"] ** 2).sqrt()
        self.weigh(self.c)

    def weigh(self, c):
        cn = self.sum("c", c * c).sqrt()
        b = torch.maximum(*[torch.where(torch.isfinite(t), t.abs(), 0.0) for t in (self.lc, self.uc)])
        bn = self.sum("r", b * b).sqrt()
        self.omega0 = torch.where((cn > 1e-10) & (bn > 1e-10), cn / bn, 1.0)

    def sum(self, which, t):
        """Per-problem sums of a row ('r') or column ('c') vector."""
        if self.B == 1:
            return t.sum().reshape(1)
        lens = self.rows if which == "r" else self.cols
        if min(lens) == max(lens):
            return t.reshape(self.B, -1).sum(1)
        return torch.segment_reduce(t, "sum", lengths=self.lens[which])

    def at(self, which, s):
        """A per-problem scalar, spread over the vector's entries."""
        if self.B == 1:
            return s
        return torch.repeat_interleave(s, self.lens[which], output_size=sum(self.rows if which == "r" else self.cols))

    @staticmethod
    def _scale(a):
        val = a.val.clone()
        dr, dc = torch.ones(a.m, dtype=F64, device=DEV), torch.ones(a.n, dtype=F64, device=DEV)
        lr, lc = torch.diff(a.rowptr), torch.diff(a.colptr)
        for k in range(11):
            how = "max" if k < 10 else "sum"
            r = torch.segment_reduce(val.abs(), how, lengths=lr)
            s = torch.segment_reduce(val[a.perm].abs(), how, lengths=lc)
            r = torch.where((lr > 0) & (r > 0), r, 1.0).sqrt()
            s = torch.where((lc > 0) & (s > 0), s, 1.0).sqrt()
            val = val / (r[a.row] * s[a.col])
            dr, dc = dr / r, dc / s
        return dr, dc, val

    @staticmethod
    def _scale_dense(a):
        dr, dc = torch.ones(a.shape[0], dtype=F64, device=DEV), torch.ones(a.shape[1], dtype=F64, device=DEV)
        for k in range(11):
            if k < 10:
                r, s = torch.maximum(a.amax(1), -a.amin(1)), torch.maximum(a.amax(0), -a.amin(0))
            else:
                r, s = torch.linalg.vector_norm(a, 1, 1), torch.linalg.vector_norm(a, 1, 0)
            r, s = torch.where(r > 0, r, 1.0).sqrt(), torch.where(s > 0, s, 1.0).sqrt()
            a.div_(r[:, None]).div_(s)
            dr, dc = dr / r, dc / s
        return dr, dc

    def _norm(self):
        """||A~||_2 by Golub-Kahan-Lanczos steps until the Ritz value moves by 1e-7."""
        j = torch.cat([torch.arange(n, device=DEV) for n in self.cols]) if self.B > 1 and min(self.cols) < max(self.cols) \
            else torch.arange(self.cols[0], device=DEV).repeat(self.B)
        v = 0.5 + _splitmix(j)
        v = v / self.at("c", self.sum("c", v * v).sqrt())
        u, beta = 0.0, torch.zeros(self.B, dtype=F64, device=DEV)
        al, be = [], []
        lam = torch.full((self.B,), math.nan, dtype=F64, device=DEV)
        while len(al) < 2000:
            u = self.mul(v) - (self.at("r", beta) * u if al else 0.0)
            alpha = self.sum("r", u * u).sqrt()
            u = u / self.at("r", torch.where(alpha > 0, alpha, 1.0))
            v = self.tmul(u) - self.at("c", alpha) * v
            beta = self.sum("c", v * v).sqrt()
            v = v / self.at("c", torch.where(beta > 0, beta, 1.0))
            al.append(alpha)
            be.append(beta)
            if len(al) % 16 == 0 or len(al) == 2:
                lam = self._stopped(torch.stack(al), torch.stack(be))
                if not torch.isnan(lam).any():
                    break
        return lam.sqrt()

    @staticmethod
    def _stopped(al, be):
        """Per problem the largest eigenvalue of B_k'B_k at the first k that
        stops (bisection with Sturm counts, all k at once), or NaN."""
        K, B = al.shape
        diag = al * al
        diag[1:] += be[:-1] ** 2
        off = al * be                                  # between k and k + 1
        ks = torch.arange(1, K + 1, device=DEV)[:, None]
        lo = torch.zeros(K, B, dtype=F64, device=DEV)
        hi = (diag + off + torch.cat([torch.zeros_like(off[:1]), off[:-1]])).amax(0).expand(K, B).clone()
        for _ in range(80):
            mid = 0.5 * (lo + hi)
            q = diag[0] - mid
            neg = q < 0
            for i in range(1, K):
                q = diag[i] - mid - off[i - 1] ** 2 / torch.where(q == 0, 1e-300, q)
                neg = neg & ((q < 0) | (ks <= i))
            lo, hi = torch.where(neg, lo, mid), torch.where(neg, mid, hi)
        lam = hi
        tiny = (al <= 1e-14 * al[:1]) | (be <= 1e-14 * al[:1])
        stop = tiny.clone()
        stop[1:] |= (lam[1:] - lam[:-1]).abs() <= 1e-7 * lam[1:].abs()
        first = torch.argmax(stop.int(), 0)
        got = lam.gather(0, first[None])[0]
        return torch.where(stop.any(0), got, math.nan)

    def start(self):
        x = torch.minimum(torch.maximum(torch.zeros_like(self.c), self.lv), self.uv)
        return x, torch.zeros_like(self.lc)

    def step(self, x, y, tau, sigma, c):
        """The PDHG point from (x, y)."""
        s = _Mul.apply(y, self.tmul, self.mul)
        xh = torch.minimum(torch.maximum(x - self.at("c", tau) * (c - s), self.lv), self.uv)
        sg = self.at("r", sigma)
        v = y / sg - _Mul.apply(2.0 * xh - x, self.mul, self.tmul)
        return xh, sg * (v - torch.minimum(torch.maximum(v, -self.uc), -self.lc))

    def kkt(self, x, y, qx=0.0):
        """(max of the relative errors, its absolute parts) of a scaled point."""
        v, xo, yo = self.v, x * self.dc, y * self.dr
        ax = self.mul(x) / self.dr
        rp = self.sum("r", (ax - torch.minimum(torch.maximum(ax, v["lc"]), v["uc"])) ** 2).sqrt()
        g = qx / self.dc + v["c"] - self.tmul(y) / self.dc
        lf, uf = torch.isfinite(v["lv"]), torch.isfinite(v["uv"])
        lam = torch.where(lf & uf, g, torch.where(lf, g.clamp(min=0.0), torch.where(uf, g.clamp(max=0.0), 0.0)))
        rd = self.sum("c", (g - lam) ** 2).sqrt()

        def support(lo, hi, w):
            return torch.where(torch.isfinite(lo), lo, 0.0) * w.clamp(min=0.0) \
                - torch.where(torch.isfinite(hi), hi, 0.0) * (-w).clamp(min=0.0)
        xqx = self.sum("c", xo * (qx / self.dc)) if torch.is_tensor(qx) else 0.0
        P = 0.5 * xqx + self.sum("c", v["c"] * xo)
        D = -0.5 * xqx + self.sum("r", support(v["lc"], v["uc"], yo)) + self.sum("c", support(v["lv"], v["uv"], lam))
        gap = (P - D).abs()
        err = torch.maximum(torch.maximum(rp / (1 + self.bnorm), rd / (1 + self.cnorm)), gap / (1 + P.abs() + D.abs()))
        return err, rp, rd, gap

    def due(self, r, t, k, w):
        """Which problems restart, and the residual they measure from next."""
        if t == 0:
            w["start"], w["prev"] = r.clone(), r.clone()
            return torch.zeros_like(r, dtype=torch.bool)
        re = (r <= 0.2 * w["start"]) | ((r <= 0.8 * w["start"]) & (r > w["prev"])) | (k >= 0.36 * t)
        w["start"], w["prev"] = torch.where(re, r, w["start"]), r.clone()
        return re

    def new_omega(self, omega, dx, dy):
        ok = (dx > 1e-10) & (dy > 1e-10)
        return torch.where(ok, torch.exp(0.5 * torch.log(dy / dx) + 0.5 * torch.log(omega)), omega)

    def solve(self, limit, eps, c=None, schedule=None):
        """Restarted Halpern PDHG from zero; eps None: exactly `limit` steps.
        schedule: a list that receives (state, omega, k, restarts, new omega) per check."""
        c = self.c if c is None else c
        x, y = self.start()
        x0, y0, omega, k, w = x, y, self.omega0, torch.zeros(self.B, dtype=F64, device=DEV), {}
        done = torch.zeros(self.B, dtype=torch.bool, device=DEV)
        outx, outy, its = torch.zeros_like(x), torch.zeros_like(y), torch.zeros(self.B, dtype=torch.int64, device=DEV)
        for t in range(limit):
            tau, sigma = self.eta / omega, self.eta * omega
            last = t == limit - 1
            if schedule is not None and t % CHECK == 0:
                schedule.append([x, y, x0, y0, omega, k, None, omega])
            xh, yh = self.step(x, y, tau, sigma, c)
            re = None
            if t % CHECK == 0 or last:
                stop = torch.full_like(done, last)
                if eps is not None:
                    stop = stop | (self.kkt(xh, yh)[0] <= eps)
                new = stop & ~done
                if bool(new.any()):
                    outx, outy = torch.where(self.at("c", new), xh, outx), torch.where(self.at("r", new), yh, outy)
                    its, done = torch.where(new, t + 1, its), done | stop
                if bool(done.all()):
                    break
                dx, dy = xh - x, yh - y
                r2 = self.sum("c", dx * dx) / tau + self.sum("r", dy * dy) / sigma + 2.0 * self.sum("r", dy * self.mul(dx))
                re = self.due(r2.clamp(min=0.0).sqrt(), t, k, w)
                omega = torch.where(re, self.new_omega(omega, self.sum("c", (xh - x0) ** 2).sqrt(),
                                                       self.sum("r", (yh - y0) ** 2).sqrt()), omega)
                if schedule is not None:
                    schedule[-1][6:] = re, omega
            x, y, x0, y0, k = self.advance(x, y, x0, y0, xh, yh, k, re)
        return outx * self.dc, outy * self.dr, its

    def advance(self, x, y, x0, y0, xh, yh, k, re):
        a, b = (k + 1) / (k + 2), 1 / (k + 2)
        xn = self.at("c", a) * (2.0 * xh - x) + self.at("c", b) * x0
        yn = self.at("r", a) * (2.0 * yh - y) + self.at("r", b) * y0
        if re is None:
            return xn, yn, x0, y0, k + 1
        rc, rr = self.at("c", re), self.at("r", re)
        return (torch.where(rc, xh, xn), torch.where(rr, yh, yn), torch.where(rc, xh, x0), torch.where(rr, yh, y0),
                torch.where(re, 0.0, k + 1))

    def unrolled_gradient(self, T, c_o, gx):
        """(x_T, y_T, dL/dc) for dL/dx_T = gx, the schedule held fixed."""
        self.v["c"], self.c = c_o.reshape(-1), c_o.reshape(-1) * self.dc
        self.weigh(self.c)
        plan = []
        x, y, _ = self.solve(T, None, schedule=plan)
        c = self.c.detach().requires_grad_()
        bar, gc = None, torch.zeros_like(c)
        for n in reversed(range(len(plan))):
            *state, omega, k, re, after = plan[n]
            leaves = [t.detach().requires_grad_() for t in state]
            xs, ys, x0, y0 = leaves
            for t in range(n * CHECK, min(T, (n + 1) * CHECK)):
                xh, yh = self.step(xs, ys, self.eta / omega, self.eta * omega, c)
                if t == T - 1:
                    break
                xs, ys, x0, y0, k = self.advance(xs, ys, x0, y0, xh, yh, k, re if t % CHECK == 0 else None)
                omega = after
            outs, bars = ([xh], [gx.reshape(-1) * self.dc]) if bar is None else ([xs, ys, x0, y0], bar)
            g = torch.autograd.grad(outs, [*leaves, c], bars, allow_unused=True)
            bar = [torch.zeros_like(l) if t is None else t for l, t in zip(leaves, g)]
            gc += 0.0 if g[4] is None else g[4]
        return x, y, gc * self.dc

    # ---- convex quadratic objectives (accelerated steps, averaged output) ----

    def set_q(self, q):
        self.q = q
        v = 0.5 + _splitmix(torch.arange(self.cols[0], device=DEV).repeat(self.B))
        v = v / self.at("c", self.sum("c", v * v).sqrt())
        lam, got = torch.zeros(self.B, dtype=F64, device=DEV), torch.zeros(self.B, dtype=torch.bool, device=DEV)
        for it in range(2000):
            w = q(v)
            new, size = self.sum("c", v * w), self.sum("c", w * w).sqrt()
            conv = (new - lam).abs() <= 1e-7 * new.abs() if it else got
            lam, got = torch.where(got, lam, new), got | conv
            if it % 8 == 7 and bool(got.all()):
                break
            v = w / self.at("c", size)
        self.norm_q = lam

    def step_qp(self, s, k, omega, q):
        x, y, xb, yb = s
        th = self.at("c", 2.0 / (k + 2))
        qv = q((1.0 - th) * xb + th * x)
        tau = 1.0 / (omega / self.eta + 2.0 * self.norm_q / (k + 1))
        s_ = _Mul.apply(y, self.tmul, self.mul)
        xn = torch.minimum(torch.maximum(x - self.at("c", tau) * (qv + self.c - s_), self.lv), self.uv)
        sg = self.at("r", self.eta * omega)
        v = y / sg - _Mul.apply(2.0 * xn - x, self.mul, self.tmul)
        yn = sg * (v - torch.minimum(torch.maximum(v, -self.uc), -self.lc))
        tr = self.at("r", 2.0 / (k + 2))
        return xn, yn, (1.0 - th) * xb + th * xn, (1.0 - tr) * yb + tr * yn

    def solve_qp(self, limit, eps, schedule=None):
        x, y = self.start()
        s, x0, y0 = (x, y, x, y), x, y
        omega, k, w = self.omega0, torch.zeros(self.B, dtype=F64, device=DEV), {}
        done = torch.zeros(self.B, dtype=torch.bool, device=DEV)
        outx, outy, its = torch.zeros_like(x), torch.zeros_like(y), torch.zeros(self.B, dtype=torch.int64, device=DEV)
        for t in range(limit):
            last = t == limit - 1
            if schedule is not None and t % CHECK == 0:
                schedule.append([s, omega, k, None, omega])
            s = self.step_qp(s, k, omega, self.q)
            if t % CHECK and not last:
                k = k + 1
                continue
            xb, yb = s[2], s[3]
            err, rp, rd, gap = self.kkt(xb, yb, self.q(xb))
            stop = torch.full_like(done, last)
            if eps is not None:
                stop = stop | (err <= eps)
            new = stop & ~done
            if bool(new.any()):
                outx, outy = torch.where(self.at("c", new), xb, outx), torch.where(self.at("r", new), yb, outy)
                its, done = torch.where(new, t + 1, its), done | stop
            if bool(done.all()):
                break
            re = self.due((omega * rp ** 2 + rd ** 2 / omega + gap ** 2).sqrt(), t, k, w)
            omega = torch.where(re, self.new_omega(omega, self.sum("c", (xb - x0) ** 2).sqrt(),
                                                   self.sum("r", (yb - y0) ** 2).sqrt()), omega)
            rc, rr = self.at("c", re), self.at("r", re)
            s = (torch.where(rc, xb, s[0]), torch.where(rr, yb, s[1]), xb, yb)
            x0, y0, k = torch.where(rc, xb, x0), torch.where(rr, yb, y0), torch.where(re, 0.0, k + 1)
            if schedule is not None:
                schedule[-1][3:] = re, omega
        return outx * self.dc, outy * self.dr, its

    def unrolled_gradient_qp(self, T, F, d, gx):
        """(x_T, dL/dc, dL/dd) for dL/dx_T = gx, the schedule held fixed."""
        plan = []
        xT, _, _ = self.solve_qp(T, None, schedule=plan)
        c_all, dd = self.c, (d.reshape(-1) * self.dc ** 2).requires_grad_()
        self.c = c_all.detach().requires_grad_()
        dc = self.dc.reshape(self.B, -1)
        Fs = F * dc[0][:, None]

        def q(v):
            vb = v.reshape(self.B, -1)
            return ((vb @ Fs) @ Fs.T).reshape(-1) + dd * v
        bar, gc, gd = None, torch.zeros_like(self.c), torch.zeros_like(dd)
        for n in reversed(range(len(plan))):
            state, omega, k, re, after = plan[n]
            leaves = [t.detach().requires_grad_() for t in state]
            s = tuple(leaves)
            for t in range(n * CHECK, min(T, (n + 1) * CHECK)):
                s = self.step_qp(s, k, omega, q)
                k = k + 1
                if t % CHECK == 0 and re is not None:
                    rc, rr = self.at("c", re), self.at("r", re)
                    s = (torch.where(rc, s[2], s[0]), torch.where(rr, s[3], s[1]), s[2], s[3])
                    k = torch.where(re, 0.0, k)
                omega = after
            outs, bars = ([s[2]], [gx.reshape(-1) * self.dc]) if bar is None else (list(s), bar)
            g = torch.autograd.grad(outs, [*leaves, self.c, dd], bars, allow_unused=True)
            bar = [torch.zeros_like(l) if t is None else t for l, t in zip(leaves, g)]
            gc += 0.0 if g[4] is None else g[4]
            gd += 0.0 if g[5] is None else g[5]
        self.c = c_all
        return xT, gc * self.dc, gd * self.dc ** 2


def _quad(d, ref):
    """The scaled Q~ v of the reference's column vectors."""
    dc = ref.dc
    if "F" in d:
        Fs, dd, B = d["F"] * dc.reshape(ref.B, -1)[0][:, None], d["d"].reshape(-1) * dc ** 2, ref.B
        return lambda v: ((v.reshape(B, -1) @ Fs) @ Fs.T).reshape(-1) + dd * v
    q = d["q"]
    if q["q_format"] == "lowrank":
        Fs, dd = q["q_factor"] * dc[:, None], q["q_diag"] * dc ** 2
        return lambda v: Fs @ (Fs.T @ v) + dd * v
    if q["q_format"] == "dense":
        return lambda v: dc * (q["q_dense"] @ (dc * v))
    n = dc.numel()
    Q = torch.sparse_csr_tensor(q["q_rowptr"].long(), q["q_colidx"].long(), q["q_val"], (n, n))
    return lambda v: dc * (Q @ (dc * v))


def exact(case, seed):
    d, kind = _inputs(case, seed), case["kind"]
    if kind == "heads":
        return dict(c=d["f"] @ d["W"], loss=(d["ct"] * d["x"]).sum(1) - d["vs"],
                    gW=(d["gc"][..., None] * d["f"]).sum((0, 1)))
    if kind == "surrogate":
        ch, ct, ws, wt = (d[k] for k in ("ch", "ct", "ws", "wt"))
        cp = ch[:, None] + 0.5 * d["Z"]
        return dict(c=2 * ch - ct, loss=-((2 * ch - ct) * wt).sum(1) + 2 * (ch * ws).sum(1) - d["zs"],
                    grad=2 * (ws - wt), cp=cp, ploss=(ch * ws).sum(1) - (cp * d["wm"]).sum(2).mean(1),
                    pgrad=ws - d["wm"].mean(1))
    ref = Reference(d, case)
    if kind in ("lp", "resolve", "dense", "qp"):
        if kind == "qp":
            ref.set_q(_quad(d, ref))
            x, y, its = ref.solve_qp(case["limit"], EPS)
        else:
            x, y, its = ref.solve(case["limit"], EPS)
        return dict(x=x, y=y, iterations=int(its[0]))
    if kind in ("grid", "ragged"):
        x, y, _ = ref.solve(10 ** 7, EPS)
        if kind == "grid":
            x, y = x.reshape(case["B"], -1), y.reshape(case["B"], -1)
        return dict(x=x, y=y)
    B, T = case["B"], case["T"]
    if kind == "learn":
        ct = d["v"]["c"]
        x, y, gc = ref.unrolled_gradient(T, d["f"] @ d["W"], ct)
        x, y, gc = x.reshape(B, -1), y.reshape(B, -1), gc.reshape(B, -1)
        return dict(x=x, y=y, loss=(ct * x).sum(1) - d["vs"], gc=gc, gW=(gc[..., None] * d["f"]).sum((0, 1)))
    ref.set_q(_quad(d, ref))
    xs, ys, _ = ref.solve_qp(10 ** 5, EPS)
    x, _, _ = ref.solve_qp(T, None)
    x, gc, gd = ref.unrolled_gradient_qp(T, d["F"], d["d"], x)
    x = x.reshape(B, -1)
    qx = (x @ d["F"]) @ d["F"].T + d["d"] * x
    return dict(xs=xs.reshape(B, -1), ys=ys.reshape(B, -1), x=x, value=(x * (0.5 * qx + d["v"]["c"])).sum(1),
                gx=qx + d["v"]["c"], gc=gc.reshape(B, -1), gd=gd.reshape(B, -1))
