"""Dense passes with fewer rows than a group of four: scaling and one iteration
against the CPU oracle, within the 1e-12 of the other step-parity tests."""

import sys

import numpy as np
import pytest

import gen
from gpu_util import rel_inf, to_np

pytestmark = pytest.mark.gpu


def _problem(m, n):
    rng = np.random.default_rng(m * 11 + n)
    a = rng.standard_normal((m, n))
    lc = rng.standard_normal(m)
    lp = gen.LP(m, n, None, None, None, rng.standard_normal(n), lc, lc + 1.0, np.zeros(n), np.full(n, 2.0), dense=a)
    return lp, [rng.standard_normal(k) for k in (n, m, n, m)]


@pytest.mark.parametrize("m,n", [(1, 40001), (2, 257), (2, 16384), (3, 1025), (3, 40000), (4, 40000), (5, 300)])
def test_fewer_rows_than_a_group(oracle_lib, m, n):
    from paper_2412_09734_amd import Solver
    print(f"case: dense {m} x {n}", file=sys.stderr, flush=True)
    lp, (x, y, x0, y0) = _problem(m, n)
    orc = oracle_lib.Oracle(lp, power_max_iters=1)
    sc = orc.scaling()
    tau, sigma = sc["eta"] / sc["omega"], sc["eta"] * sc["omega"]
    ref = orc.lp_step(x, y, x0, y0, 5, tau, sigma)
    with Solver.from_lp(lp, power_max_iters=1) as s:
        gs = s.scaling()
        assert rel_inf(to_np(gs["dc"]), sc["dc"]) <= 1e-12 and rel_inf(to_np(gs["dr"]), sc["dr"]) <= 1e-12
        got = [*s.debug_step(x, y, x0, y0, 5, tau, sigma), *s.debug_plain_step(x, y, x0, y0, 5, tau, sigma)]
    for g, r in zip(got, [*ref, *ref[2:]]):
        assert rel_inf(to_np(g), r) <= 1e-12
    with Solver.from_lp(lp, iteration_limit=20000) as s:   # one norm step is too few for a solve
        assert s.solve()[2]["status_name"] == "optimal"
