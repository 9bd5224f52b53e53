"""Low-rank QPs with more partial sums of F'v than a workgroup adds by itself (512,
131,072 columns): 130 iterations from the start against the CPU oracle. Tolerance:
130 steps of rounding in sums of up to 300,000 products in another order, 1e-10 of
their absolute terms, as in the other QP tests."""

import sys

import numpy as np
import pytest

import gen
from gpu_util import rel_inf, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rank", [(131072, 3), (131073, 8), (140001, 1), (200003, 17), (300000, 32)])
def test_iterations(oracle_lib, n, rank):
    from paper_2412_09734_amd import Solver
    print(f"case: low-rank QP n={n} rank={rank}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(n + rank)
    m = 40
    cols = np.sort(rng.choice(n, (m, 30), replace=False), axis=1)
    val = rng.standard_normal((m, 30))
    x = rng.random(n)
    ax = (val * x[cols]).sum(1)
    lp = gen.LP(m, n, (30 * np.arange(m + 1)).astype(np.int32), cols.reshape(-1).astype(np.int32), val.reshape(-1),
                rng.standard_normal(n), ax, ax + 0.5, np.zeros(n), np.full(n, 2.0), q_kind="lowrank",
                q_factor=rng.standard_normal((n, rank)) / np.sqrt(n), q_diag=rng.uniform(0.01, 0.1, n))
    opts = dict(eps=1e-13, iteration_limit=130)
    xo, yo, ro = oracle_lib.Oracle(lp, **opts).solve()
    with Solver.from_lp(lp, **opts) as s:
        xs, ys, rs = s.solve()
    assert rs["iterations"] == ro["iterations"] and rs["restarts"] == ro["restarts"]
    assert rel_inf(to_np(xs), xo) <= 1e-10 and rel_inf(to_np(ys), yo) <= 1e-10
