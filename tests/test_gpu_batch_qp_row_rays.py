"""Batched QPs with one constraint row: the rays of infeasible instances checked by
themselves on the host, and step sizes equal to the oracle's, so that the
comparisons with its trajectory apply."""

import sys

import numpy as np
import pytest

import gen
from gpu_util import to_np
from test_gpu_batch_qp_row import _batch, _oracle, _problem

pytestmark = pytest.mark.gpu

EPS = 1e-8   # the default certificate tolerances


@pytest.mark.parametrize("n,rank,every", [(1, 1, 1), (63, 8, 1), (65, 9, 2), (256, 16, 1), (257, 17, 3),
                                          (512, 24, 1), (511, 32, 1), (513, 25, 1), (1024, 32, 1), (1025, 3, 1)])
def test_step_sizes(oracle_lib, n, rank, every):
    from paper_2412_09734_amd.solver import BatchSolver
    p = _problem(n, rank, 2, seed=100 + n, every=every)
    with BatchSolver.from_shared(_batch(p), iteration_limit=1) as bs:
        res = bs.solve()[2]
    for b in range(2):
        assert abs(_oracle(oracle_lib, p, b).scaling()["eta"] / res[b]["eta"] - 1.0) <= 1e-12


def _bound_terms(g, lv, uv):
    """lam, the bound-cone part of the reduced costs g, and the bounds' objective."""
    lf, uf = np.isfinite(lv), np.isfinite(uv)
    lam = np.where(lf & uf, g, np.where(lf, np.maximum(g, 0.0), np.where(uf, np.minimum(g, 0.0), 0.0)))
    obj = np.where(lf, np.where(lf, lv, 0.0) * np.maximum(lam, 0.0), 0.0) - \
        np.where(uf, np.where(uf, uv, 0.0) * np.maximum(-lam, 0.0), 0.0)
    return lam, obj.sum()


# one, two columns per thread, 512 threads; a ray is the difference of close points
# over a scale: its sums are right to 1e-6
@pytest.mark.parametrize("n,rank", [(70, 5), (300, 9), (700, 26)])
@pytest.mark.parametrize("kind", ["primal", "dual"])
def test_rays(kind, n, rank):
    from paper_2412_09734_amd.solver import BatchSolver
    print(f"case: one row, {kind} infeasible, n={n} rank={rank}", file=sys.stderr, flush=True)
    p = _problem(n, rank, 2, seed=9, every=2)
    a = np.zeros(n)
    a[p["colidx"]] = p["val"]
    last = n - 1 if a[n - 1] == 0.0 else n - 2
    if kind == "primal":
        p["uv"] = np.full(n, 0.2 / n)         # the budget cannot be met
    else:
        p["F"][last] = 0.0                    # a column that is linear, unbounded, not in the row
        p["d"][:, last] = 0.0
        p["c"][:, last] = -1.0
        p["uv"][last] = np.inf
    with BatchSolver.from_shared(_batch(p), iteration_limit=200000) as bs:
        x, y, res = bs.solve()
    for b in range(2):
        xb, yb = to_np(x[b]), to_np(y[b])
        assert res[b]["status_name"] == ("primal_infeasible" if kind == "primal" else "dual_infeasible")
        if kind == "primal":
            g = -a * yb[0]
            lam, obj = _bound_terms(g, p["lv"], p["uv"])
            obj += p["lc"][0] * max(yb[0], 0.0) - p["uc"][0] * max(-yb[0], 0.0)
            assert abs(obj - 1.0) <= 1e-6 and np.abs(g - lam).max() <= EPS * (1.0 + 1e-6)
        else:
            assert abs(p["c"][b] @ xb + 1.0) <= 1e-6
            out = np.maximum(np.where(np.isfinite(p["lv"]), -xb, 0.0), np.where(np.isfinite(p["uv"]), xb, 0.0))
            qx = p["F"] @ (p["F"].T @ xb) + p["d"][b] * xb
            assert max(out.max(), abs(a @ xb), np.abs(qx).max()) <= EPS * (1.0 + 1e-6)
