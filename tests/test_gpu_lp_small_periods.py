"""Small LPs with check periods longer than one launch of the one-workgroup solve
takes (4,096 iterations): split periods against the multi-kernel iteration. Up to
21,000 nonexpansive steps of rounding 1e-15 of the iterates' size, times the
spread of the scaling (below 1e2): 1e-8."""

import sys

import numpy as np
import pytest

import gen
from gpu_util import rel_inf, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("check_every,limit", [(4096, 4097), (4097, 4098), (4097, 8300), (4098, 4099), (4098, 9000),
                                               (5000, 5000), (8194, 8200), (8193, 20000), (100000, 9000), (20000, 21000),
                                               (2000, 4500), (1366, 4200)])
def test_long_periods(check_every, limit):
    from paper_2412_09734_amd import Solver
    print(f"case: small LP, check every {check_every}, limit {limit}", file=sys.stderr, flush=True)
    lp = gen.planted_sparse_lp(60, 130, density=0.05, seed=8)
    out = []
    for kw in ({}, dict(timing_chunk=1 << 30, use_graph=0)):
        with Solver.from_lp(lp, eps=1e-300, check_every=check_every, iteration_limit=limit, eps_primal_infeasible=0.0,
                            eps_dual_infeasible=0.0, **kw) as s:
            x, y, r = s.solve()
            out.append((to_np(x), to_np(y), r))
    (x, y, r), (x0, y0, r0) = out
    assert (r["iterations"], r["restarts"], r["status"]) == (r0["iterations"], r0["restarts"], r0["status"])
    assert r["iterations"] == limit
    assert rel_inf(x, x0) <= 1e-8 and rel_inf(y, y0) <= 1e-8


def test_a_long_period_ends_at_its_first_check():
    """Optimal at the warm start: the rest of the period's launches do nothing."""
    from paper_2412_09734_amd import Solver
    lp = gen.planted_sparse_lp(60, 130, density=0.05, seed=8)
    with Solver.from_lp(lp) as s:
        x, y, _ = s.solve()
    with Solver.from_lp(lp, check_every=50000, eps=2e-4) as s:
        x2, y2, r = s.solve(x_init=x, y_init=y)
        first = r["iterations"]
        x3, y3, r3 = s.solve()
    assert first == 1 and r["status_name"] == "optimal"
    assert r3["status_name"] == "optimal" and r3["iterations"] in (50001, 100001)
