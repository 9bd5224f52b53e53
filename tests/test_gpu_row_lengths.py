"""GPU parity of one iteration where the layout of the sparse products changes:
row lengths at the edges of the lane groups and of the unrolled entry groups,
and matrices on both sides of the row count from which a thread sums a row."""

import sys

import numpy as np
import pytest

import gen
from gpu_util import rel_inf, to_np

pytestmark = pytest.mark.gpu

STEP_TOL = 1e-12   # as in the other step-parity tests: FP64 sums in another order

EDGES = [0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512,
         513, 1023, 1024, 1025, 2047, 2048, 2049]


def _lp(m, n, degrees, seed):
    """Columns of the given lengths (cycled), rows uniform per column."""
    rng = np.random.default_rng(seed)
    deg = np.minimum(np.resize(degrees, n), m)
    rows = np.concatenate([rng.choice(m, size=d, replace=False) for d in deg])
    cols = np.repeat(np.arange(n), deg)
    order = np.lexsort((cols, rows))
    rowptr = np.zeros(m + 1, dtype=np.int32)
    np.cumsum(np.bincount(rows, minlength=m), out=rowptr[1:])
    val = rng.standard_normal(len(rows))
    lc = rng.standard_normal(m)
    return gen.LP(m, n, rowptr, cols[order].astype(np.int32), val[order], rng.standard_normal(n), lc, lc + 1.0,
                  np.zeros(n), np.full(n, 2.0))


@pytest.mark.parametrize("m,n,degrees", [
    (2100, 66, EDGES), (2100, 3, [2049, 65, 5]), (130, 700, [3, 70]),
    (49152, 150, EDGES), (49153, 150, EDGES), (60, 49200, [1, 2, 3]), (50000, 60000, [0, 4, 20])])
def test_step_parity_row_lengths(oracle_lib, m, n, degrees):
    from paper_2412_09734_amd import Solver
    print(f"case: row lengths, {m} x {n}", file=sys.stderr, flush=True)
    lp = _lp(m, n, degrees, seed=m + n)
    orc = oracle_lib.Oracle(lp, power_max_iters=1)
    sc = orc.scaling()
    rng = np.random.default_rng(5)
    x, x0 = rng.standard_normal(n), rng.standard_normal(n)
    y, y0 = rng.standard_normal(m), rng.standard_normal(m)
    tau, sigma = sc["eta"] / sc["omega"], sc["eta"] * sc["omega"]
    ref = orc.lp_step(x, y, x0, y0, 3, tau, sigma)
    with Solver.from_lp(lp, power_max_iters=1) as s:
        for nm, g, r in zip(("xhat", "yhat", "xnew", "ynew"), s.debug_step(x, y, x0, y0, 3, tau, sigma), ref):
            assert rel_inf(to_np(g), r) <= STEP_TOL, nm
        for nm, g, r in zip(("xnew", "ynew"), s.debug_plain_step(x, y, x0, y0, 3, tau, sigma), ref[2:]):
            assert rel_inf(to_np(g), r) <= STEP_TOL, nm
