"""Dense passes with infinite entries in the gathered vectors: one iteration against
the CPU oracle, within the 1e-12 of the other step-parity tests."""

import sys

import numpy as np
import pytest

import gen
from gpu_util import to_np

pytestmark = pytest.mark.gpu


def _problem(m, n):
    rng = np.random.default_rng(m * 11 + n)
    a = rng.standard_normal((m, n))
    lc = rng.standard_normal(m)
    lp = gen.LP(m, n, None, None, None, rng.standard_normal(n), lc, lc + 1.0, np.zeros(n), np.full(n, 2.0), dense=a)
    return lp, [rng.standard_normal(k) for k in (n, m, n, m)]


@pytest.mark.parametrize("m,n", [(3, 70), (9, 130), (100, 65), (700, 1500), (1030, 3001), (2100, 70)])
def test_infinite_entries(oracle_lib, m, n):
    """An infinite last entry of y (of x_ext): the sums of all columns (rows) are
    infinities of the entry's sign, also where the last rows (columns) of a tile
    are clamped to it."""
    from paper_2412_09734_amd import Solver
    print(f"case: dense {m} x {n}, infinite entries", file=sys.stderr, flush=True)
    lp, (x, y, x0, y0) = _problem(m, n)
    orc = oracle_lib.Oracle(lp, power_max_iters=1)
    sc = orc.scaling()
    tau, sigma = sc["eta"] / sc["omega"], sc["eta"] * sc["omega"]
    with Solver.from_lp(lp, power_max_iters=1) as s:
        y[-1] = np.inf
        ref, got = orc.lp_step(x, y, x0, y0, 5, tau, sigma)[0], to_np(s.debug_step(x, y, x0, y0, 5, tau, sigma)[0])
        assert np.all(np.abs(got - ref) <= 1e-12 * (1.0 + np.abs(ref)))
        y[-1], x[-1] = 0.5, -np.inf     # x^ is at a bound, x_ext = 2 x^ - x infinite
        ref, got = orc.lp_step(x, y, x0, y0, 5, tau, sigma)[1], to_np(s.debug_step(x, y, x0, y0, 5, tau, sigma)[1])
        assert np.isinf(ref).all() and np.array_equal(got, ref)
