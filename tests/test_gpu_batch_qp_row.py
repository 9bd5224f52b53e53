"""GPU parity of the batched QP kernels for one constraint row at the edges of
their column and rank blocks, with rows that miss columns, replayed schedules
and certificates, against the CPU oracle. Tolerances are those of the other
batched QP tests: unrolled points 1e-10, reverse pass 1e-9, equal iterations."""

import sys
from types import SimpleNamespace

import numpy as np
import pytest

import gen
from gpu_util import rel_inf, to_np

pytestmark = pytest.mark.gpu


def _problem(n, rank, B, seed, every=1):
    """Portfolio QPs whose budget row holds every `every`-th column."""
    p = gen.portfolio_qp_batch(batch=B, n=n, rank=rank, seed=seed)
    rng = np.random.default_rng(seed)
    cols = np.arange(0, n, every, dtype=np.int32)
    p.update(rowptr=np.array([0, len(cols)], dtype=np.int32), colidx=cols,
             val=rng.uniform(0.5, 1.5, len(cols)), uv=np.full(n, max(0.1, 8.0 / n)))
    return p


def _batch(p):
    B = p["c"].shape[0]
    return SimpleNamespace(m=1, n=p["n"], rowptr=p["rowptr"], colidx=p["colidx"], val=p["val"], c=p["c"],
                           lc=np.tile(p["lc"], (B, 1)), uc=np.tile(p["uc"], (B, 1)),
                           lv=np.tile(p["lv"], (B, 1)), uv=np.tile(p["uv"], (B, 1)),
                           q_factor=p["F"], q_diag=p["d"])


def _oracle(lib, p, b, **opts):
    return lib.Oracle(gen.LP(1, p["n"], p["rowptr"], p["colidx"], p["val"], p["c"][b].copy(), p["lc"].copy(),
                             p["uc"].copy(), p["lv"].copy(), p["uv"].copy(), q_kind="lowrank", q_factor=p["F"],
                             q_diag=p["d"][b].copy()), **opts)


@pytest.mark.parametrize("n,rank,every", [(1, 1, 1), (63, 8, 1), (65, 9, 2), (256, 16, 1), (257, 17, 3),
                                          (512, 24, 1), (511, 32, 1), (513, 25, 1), (1024, 32, 1), (1025, 3, 1)])
def test_one_row_batches(oracle_lib, n, rank, every):
    from paper_2412_09734_amd.solver import BatchSolver
    print(f"case: one constraint row, n={n} rank={rank} every={every}", file=sys.stderr, flush=True)
    B, T = 3, 131
    p = _problem(n, rank, B, seed=100 + n, every=every)
    rng = np.random.default_rng(3)
    gx, gy = rng.standard_normal((B, n)), rng.standard_normal((B, 1))
    def run(**kw):
        with BatchSolver.from_shared(_batch(p), **kw) as bs:
            x, y = bs.unrolled(T)
            g = bs.backward(gx, gy)
            xr, yr = bs.unrolled(T, replay=True)
            gr = bs.backward(gx, gy)
            xs, ys, res = bs.solve()
        assert np.array_equal(to_np(x), to_np(xr)) and np.array_equal(to_np(y), to_np(yr))
        assert all(np.array_equal(to_np(u), to_np(v)) for u, v in zip(g, gr))
        return [to_np(t) for t in (x, y, *g, xs, ys)], res
    (x, y, gc, glc, guc, gd, xs, ys), res = run()
    gen_out, gen_res = run(threads=128)      # the general kernels
    for b in range(B):
        refs = [(gen_out[0][b], gen_out[1][b], gen_out[2][b], gen_out[3][b] + gen_out[4][b], gen_out[5][b],
                 gen_out[6][b], gen_res[b])]
        o = _oracle(oracle_lib, p, b)
        # the norm estimate of a matrix with one row rests on a residual that
        # is zero up to rounding: where the step sizes agree, the oracle's
        # trajectory is the reference too
        if abs(o.scaling()["eta"] / res[b]["eta"] - 1.0) <= 1e-12:
            xo, yo, sr, sw = o.unrolled_qp(T)
            go = o.backward_qp(T, sr, sw, gx[b], gy[b])
            xso, yso, ro = o.solve()
            refs.append((xo, yo, go[0], go[1] + go[2], go[3], xso, ro))
        for xo, yo, gco, gro, gdo, xso, ro in refs:
            assert rel_inf(x[b], xo) <= 1e-10 and rel_inf(y[b], yo) <= 1e-10
            assert rel_inf(gc[b], gco) <= 1e-9 and rel_inf(gd[b], gdo) <= 1e-9
            # an equality row: rounding picks the side that takes its sensitivity
            assert rel_inf(glc[b] + guc[b], gro) <= 1e-9
            assert res[b]["iterations"] == ro["iterations"] and res[b]["status"] == ro["status"]
            assert rel_inf(xs[b], xso) <= 1e-9


@pytest.mark.parametrize("kind", ["primal", "dual"])
def test_one_row_certificates(oracle_lib, kind):
    from paper_2412_09734_amd.solver import BatchSolver
    print(f"case: one constraint row, {kind} infeasible", file=sys.stderr, flush=True)
    p = _problem(70, 5, 2, seed=9, every=2)
    if kind == "primal":
        p["uv"] = np.full(70, 0.2 / 70)        # the budget cannot be met
    else:
        p["F"][69] = 0.0                       # column 69: linear, unbounded, not in the row
        p["d"][:, 69] = 0.0
        p["c"][:, 69] = -1.0
        p["uv"][69] = np.inf
    with BatchSolver.from_shared(_batch(p), iteration_limit=60000) as bs:
        x, y, res = bs.solve()
    for b in range(2):
        xo, yo, ro = _oracle(oracle_lib, p, b, iteration_limit=60000).solve()
        assert res[b]["status"] == ro["status"]
        assert abs(res[b]["iterations"] - ro["iterations"]) <= 64
        if res[b]["iterations"] == ro["iterations"]:
            assert rel_inf(to_np(y[b]) if kind == "primal" else to_np(x[b]), yo if kind == "primal" else xo) <= 1e-6
