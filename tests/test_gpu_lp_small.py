"""The one-workgroup solve of small LPs against the multi-kernel iteration
(timing_chunk >= 0 asks for it) and the CPU oracle: sizes on both sides of its
task counts, row lengths past its registers, limits around the check period.
Both run the same formulas in FP64, so after a few hundred iterations the points
agree to 1e-10 and the counts exactly, as in the other solve tests."""

import sys

import numpy as np
import pytest

import gen
from gpu_util import rel_inf, to_np

pytestmark = pytest.mark.gpu


def _say(*a):
    print("case:", *a, file=sys.stderr, flush=True)


def _columns(m, n, degrees, seed):
    """Boxed LP whose columns have the given lengths (cycled)."""
    rng = np.random.default_rng(seed)
    deg = np.minimum(np.resize(degrees, n), m)
    rows = np.concatenate([rng.choice(m, size=d, replace=False) for d in deg])
    cols = np.repeat(np.arange(n), deg)
    order = np.lexsort((cols, rows))
    rowptr = np.zeros(m + 1, dtype=np.int32)
    np.cumsum(np.bincount(rows, minlength=m), out=rowptr[1:])
    val = rng.standard_normal(len(rows))
    x = rng.random(n)
    ax = np.zeros(m)
    np.add.at(ax, rows, val[np.argsort(order)] * x[cols])
    return gen.LP(m, n, rowptr, cols[order].astype(np.int32), val, rng.standard_normal(n), ax - 0.5,
                  np.where(rng.random(m) < 0.5, ax - 0.5, np.inf), np.zeros(n), np.full(n, 2.0))


def _pair(lp, **opts):
    from paper_2412_09734_amd import Solver
    out = []
    for kw in ({}, {"timing_chunk": 1 << 30}):
        with Solver.from_lp(lp, **opts, **kw) as s:
            x, y, r = s.solve()
            x2, y2, r2 = s.solve(x_init=x, y_init=y)
            out.append((to_np(x), to_np(y), r, to_np(x2), to_np(y2), r2))
    return out


@pytest.mark.parametrize("m,n,degrees", [
    (1, 1, [1]), (3, 2, [3]), (64, 64, [4]), (65, 130, [4, 5]), (700, 64, [300, 513, 2, 700]), (256, 1024, [4]),
    (300, 1030, [3, 4]), (200, 2048, [2]), (500, 1000, [8, 9]), (900, 2400, [3]), (1100, 2400, [4]), (40, 3000, [1])])
def test_small_matches_launches_and_oracle(oracle_lib, m, n, degrees):
    _say(f"small LP {m} x {n}")
    lp = _columns(m, n, degrees, seed=m + n)
    a, b = _pair(lp, iteration_limit=200, eps=1e-9)
    for u, v in zip(a, b):
        if isinstance(u, dict):
            assert (u["iterations"], u["restarts"], u["status"]) == (v["iterations"], v["restarts"], v["status"])
            assert abs(u["kkt_rel"] - v["kkt_rel"]) <= 1e-10
        else:
            assert rel_inf(u, v) <= 1e-10
    xo, yo, ro = oracle_lib.Oracle(lp, iteration_limit=200, eps=1e-9).solve()
    assert a[2]["iterations"] == ro["iterations"] and a[2]["restarts"] == ro["restarts"]
    assert rel_inf(a[0], xo) <= 1e-9 and rel_inf(a[1], yo) <= 1e-9


@pytest.mark.parametrize("limit", [1, 2, 63, 64, 65, 66, 128, 129, 448, 449, 450, 512, 513, 1025])
def test_small_limits(limit):
    _say(f"small LP, iteration limit {limit}")
    a, b = _pair(gen.planted_sparse_lp(seed=3), iteration_limit=limit, eps=1e-14)
    assert a[2]["iterations"] == b[2]["iterations"] == limit
    assert a[2]["status_name"] == b[2]["status_name"] == "iteration_limit"
    assert rel_inf(a[0], b[0]) <= 1e-10 and rel_inf(a[1], b[1]) <= 1e-10


def test_small_cadence_time_limit_and_verbose(capfd):
    _say("small LP, check cadence 7, time limit, verbose")
    lp = gen.planted_sparse_lp(seed=4)
    a, b = _pair(lp, check_every=7)
    assert a[2]["iterations"] == b[2]["iterations"] and rel_inf(a[0], b[0]) <= 1e-10
    a, b = _pair(lp, verbose=1, display_frequency=1)
    assert a[2]["iterations"] == b[2]["iterations"]
    checks = capfd.readouterr().err.count("pdhg t=")
    # a line per check of each of the four solves
    assert checks >= sum((r["iterations"] - 1) // 64 + 1 for r in (a[2], a[5], b[2], b[5]))
    from paper_2412_09734_amd import Solver
    with Solver.from_lp(lp, time_limit_s=1e-6, eps=1e-15) as s:
        r = s.solve()[2]
    assert r["status_name"] == "time_limit" and r["iterations"] % 64 == 1
