"""GPU parity of the plain rAPDHG iteration for each storage of Q at the edges
of its blocks (ranks around the fused limit, rows of Q past one lane group,
sizes around a workgroup), with restarts, against the CPU oracle: one iteration
within 1e-12, 130 iterations with equal restarts and points within 1e-9."""

import sys

import numpy as np
import pytest

import gen
from gpu_util import rel_inf, to_np

pytestmark = pytest.mark.gpu


def _qp(m, n, fmt, rank, seed):
    rng = np.random.default_rng(seed)
    lp = gen.planted_sparse_lp(m, n, density=min(1.0, 4.0 / max(m, 4)), seed=seed) if m else None
    if lp is None:
        lp = gen.LP(0, n, np.zeros(1, dtype=np.int32), np.zeros(0, dtype=np.int32), np.zeros(0),
                    rng.standard_normal(n), np.zeros(0), np.zeros(0), np.zeros(n), np.full(n, 3.0))
    lp.uv = np.full(n, 5.0)
    if fmt == "lowrank":
        lp.q_kind, lp.q_factor, lp.q_diag = "lowrank", 0.2 * rng.standard_normal((n, rank)), rng.uniform(0.01, 0.1, n)
        return lp, lp
    g = rng.standard_normal((n, rank)) * 0.3 * (rng.random((n, rank)) < 0.5)
    q = g @ g.T + np.diag(rng.uniform(0.05, 0.2, n))
    lp.q_kind = "csr"
    lp.q_rowptr, lp.q_colidx, lp.q_val = gen.csr_from_dense(q)
    if fmt == "csr":
        return lp, lp
    from types import SimpleNamespace
    d = SimpleNamespace(**{k: getattr(lp, k) for k in ("m", "n", "rowptr", "colidx", "val", "c", "lc", "uc", "lv", "uv")})
    d.q_kind, d.q_dense = "dense", q
    return d, lp


@pytest.mark.parametrize("m,n,fmt,rank", [
    (20, 1, "lowrank", 1), (20, 63, "lowrank", 8), (20, 257, "lowrank", 9), (30, 512, "lowrank", 32),
    (30, 300, "lowrank", 33), (0, 300, "lowrank", 5), (700, 9000, "lowrank", 17), (20, 5, "csr", 2),
    (20, 64, "csr", 8), (30, 513, "csr", 3), (0, 33, "csr", 4), (20, 1, "dense", 1), (20, 65, "dense", 4),
    (30, 511, "dense", 6), (30, 520, "dense", 6), (0, 40, "dense", 3)])
def test_qp_step_and_run(oracle_lib, m, n, fmt, rank):
    from paper_2412_09734_amd import Solver
    print(f"case: QP {m} x {n}, Q {fmt} rank {rank}", file=sys.stderr, flush=True)
    gpu, ref = _qp(m, n, fmt, rank, seed=n + rank)
    orc = oracle_lib.Oracle(ref, iteration_limit=130, eps=1e-14)
    rng = np.random.default_rng(1)
    x, xb, y, yb = rng.random(n), rng.random(n), rng.standard_normal(m), rng.standard_normal(m)
    with Solver.from_lp(gpu, iteration_limit=130, eps=1e-14) as s:
        for k in (0, 7):
            got = s.debug_qp_step(x, y, xb, yb, k, 0.7)
            want = orc.qp_step(x, y, xb, yb, k, 0.7)
            for nm, g, r in zip(("x", "y", "xbar", "ybar"), got, want):
                assert rel_inf(to_np(g), r) <= 1e-12, (nm, k)
        xs, ys, r = s.solve()
        x2, y2, r2 = s.solve(x_init=xs, y_init=ys if m else None)
    xo, yo, ro = orc.solve()
    assert (r["iterations"], r["restarts"]) == (ro["iterations"], ro["restarts"])
    assert rel_inf(to_np(xs), xo) <= 1e-9 and rel_inf(to_np(ys), yo) <= 1e-9
    assert r2["kkt_rel"] <= max(1e-10, 10 * r["kkt_rel"])
