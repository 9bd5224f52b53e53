"""GPU parity of the dense passes at the edges of their tiles, row groups,
splits and dispatch rules: scaling and one iteration against the CPU oracle,
within the 1e-12 of the other step-parity tests."""

import sys

import numpy as np
import pytest

import gen
from gpu_util import rel_inf, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [
    (1, 1), (1, 70), (3, 2), (4, 17), (5, 63), (6, 64), (7, 65), (16, 255), (17, 257), (63, 1023), (64, 1024),
    (65, 1030), (129, 4), (257, 513), (1025, 40), (2047, 70), (2048, 70), (2049, 70), (2049, 3000), (2, 16383),
    (5, 16384), (9, 40000), (700, 1500), (515, 33000)])
def test_dense_shape_step(oracle_lib, m, n):
    from paper_2412_09734_amd import Solver
    print(f"case: dense {m} x {n}, scaling and one step", file=sys.stderr, flush=True)
    rng = np.random.default_rng(m * 7 + n)
    a = rng.standard_normal((m, n))
    lc = rng.standard_normal(m)
    lp = gen.LP(m, n, None, None, None, rng.standard_normal(n), lc, lc + 1.0, np.zeros(n), np.full(n, 2.0), dense=a)
    orc = oracle_lib.Oracle(lp, power_max_iters=1)
    sc = orc.scaling()
    x, x0 = rng.standard_normal(n), rng.standard_normal(n)
    y, y0 = rng.standard_normal(m), rng.standard_normal(m)
    tau, sigma = sc["eta"] / sc["omega"], sc["eta"] * sc["omega"]
    ref = orc.lp_step(x, y, x0, y0, 5, tau, sigma)
    with Solver.from_lp(lp, power_max_iters=1) as s:
        gs = s.scaling()
        assert rel_inf(to_np(gs["dc"]), sc["dc"]) <= 1e-12 and rel_inf(to_np(gs["dr"]), sc["dr"]) <= 1e-12
        for nm, g, r in zip(("xhat", "yhat", "xnew", "ynew"), s.debug_step(x, y, x0, y0, 5, tau, sigma), ref):
            assert rel_inf(to_np(g), r) <= 1e-12, nm
        for nm, g, r in zip(("xnew", "ynew"), s.debug_plain_step(x, y, x0, y0, 5, tau, sigma), ref[2:]):
            assert rel_inf(to_np(g), r) <= 1e-12, nm
