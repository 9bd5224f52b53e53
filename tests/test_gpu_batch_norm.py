"""The batched norm estimate: eigenvalues are found eight steps at a time by
separate waves, from a bracket around the last one. Step size and step count
against the CPU oracle for step limits around those groups and past the part of
the tridiagonal kept on chip, for every setup width."""

import sys

import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


def _path(nodes):
    """Flow along a path (a slowly converging norm estimate)."""
    ar = np.arange(nodes - 1)
    rows, cols = np.concatenate([ar, ar + 1]), np.concatenate([ar, ar])
    val = np.concatenate([np.ones(nodes - 1), -np.ones(nodes - 1)])
    order = np.lexsort((cols, rows))
    rowptr = np.zeros(nodes + 1, dtype=np.int32)
    np.cumsum(np.bincount(rows, minlength=nodes), out=rowptr[1:])
    b = np.zeros(nodes)
    b[0], b[-1] = 1.0, -1.0
    return gen.LP(nodes, nodes - 1, rowptr, cols[order].astype(np.int32), val[order], np.ones(nodes - 1), b, b.copy(),
                  np.zeros(nodes - 1), np.full(nodes - 1, 2.0))


@pytest.mark.parametrize("nodes", [40, 600, 2100])      # 256, 512 and 1,024 threads
@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 8, 9, 17, 255, 256, 257, 300])
def test_norm_steps(oracle_lib, nodes, steps):
    from paper_2412_09734_amd.solver import BatchSolver
    print(f"case: norm estimate, {nodes} nodes, at most {steps} steps", file=sys.stderr, flush=True)
    lps = [_path(nodes), _path(nodes - 7)]
    opts = dict(power_max_iters=steps, power_tol=1e-12, iteration_limit=2)
    with BatchSolver.from_lps(lps, **opts) as bs:
        res = bs.solve()[2]
    for lp, r in zip(lps, res):
        sc = oracle_lib.Oracle(lp, **opts).scaling()
        assert abs(r["eta"] - sc["eta"]) <= 1e-10 * sc["eta"]
        assert abs(r["power_iters"] - sc["power_iters"]) <= (0 if sc["power_iters"] == steps else 1)
