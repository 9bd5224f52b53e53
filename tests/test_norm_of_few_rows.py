"""Norm estimates of matrices with so few rows that the Krylov space closes: the
step size times the norm of the scaled matrix is the safety factor 0.998, to the
rounding of some thousand squares, also where the last residual is exactly 0 (as
it is for about one length in fifty of a single row)."""

import sys

import numpy as np
import pytest

import gen

SIZES = [(1, 4 * k + 3) for k in range(1, 40)] + [(1, 3001), (1, 5000), (1, 16384), (1, 40001), (2, 700), (3, 1025)]


def _lp(m, n, dense=False, ones=False):
    rng = np.random.default_rng(m * 11 + n)
    a = np.ones((m, n)) if ones else rng.standard_normal((m, n))
    lc = rng.standard_normal(m)
    v = (rng.standard_normal(n), lc, lc + 1.0, np.zeros(n), np.full(n, 2.0))
    if dense:
        return gen.LP(m, n, None, None, None, *v, dense=a), a
    return gen.LP(m, n, *gen.csr_from_dense(a), *v), a


def _ratio(a, dr, dc, eta):
    return eta * np.linalg.norm(np.asarray(dr)[:, None] * a * np.asarray(dc), 2)


@pytest.mark.parametrize("ones", [False, True])
def test_oracle(oracle_lib, ones):
    for m, n in SIZES:
        lp, a = _lp(m, n, ones=ones)
        sc = oracle_lib.Oracle(lp).scaling()
        assert abs(_ratio(a, sc["dr"], sc["dc"], sc["eta"]) - 0.998) <= 1e-10, (m, n)


@pytest.mark.gpu
@pytest.mark.parametrize("ones", [False, True])
@pytest.mark.parametrize("form", ["sparse", "dense", "batch"])
def test_gpu(form, ones):
    from paper_2412_09734_amd.solver import BatchSolver, Solver
    print(f"case: norms of few rows, {form}", file=sys.stderr, flush=True)
    for m, n in SIZES:
        lp, a = _lp(m, n, dense=form == "dense", ones=ones)
        with Solver.from_lp(lp) as s:
            sc = s.scaling()
        dr, dc, eta = sc["dr"].cpu().numpy(), sc["dc"].cpu().numpy(), sc["eta"]
        if form == "batch":
            # the scaling is the single solver's to rounding, the norm is its own
            one = dict(shared_a=True, batch=1, m=m, n=n, rowptr=lp.rowptr, colidx=lp.colidx, val=lp.val, c=lp.c,
                       lc=lp.lc, uc=lp.uc, lv=lp.lv, uv=lp.uv, iteration_limit=1)
            with BatchSolver(**one) as bs:
                eta = bs.solve()[2][0]["eta"]
        assert abs(_ratio(a, dr, dc, eta) - 0.998) <= 1e-10, (m, n)
