"""The on-chip batched solve at every number of columns and rows per thread, one
and two (register pairs, LDS pairs, streamed ones) up to eight (streamed), against
the memory-resident kernel, which an instance of more than 8,192 columns in the
batch sends all of them to; ragged batches, the same instances on a shared
matrix, and certificates against the oracle. Also the launch that off-chip
batches start with, against the oracle."""

import sys

import numpy as np
import pytest

import gen
from gpu_util import rel_inf, to_np

pytestmark = pytest.mark.gpu

# row lengths around the pairs kept in registers (12, 16, 24, 28 entries) and groups of four pairs
LENGTHS = np.array([0, 1, 2, 3, 4, 7, 8, 9, 11, 12, 13, 16, 17, 23, 24, 25, 28, 29, 36, 37, 70])
KEYS = ("c", "lc", "uc", "lv", "uv")


def _say(*a):
    print("case:", *a, file=sys.stderr, flush=True)


def _instance(m, n, rng, longest=70):
    lens = np.minimum(rng.choice(LENGTHS[LENGTHS <= longest], m), n)
    cols = [np.sort(rng.choice(n, k, replace=False)) for k in lens]
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ci = np.concatenate(cols + [np.empty(0, np.int64)]).astype(np.int64)
    va = rng.standard_normal(len(ci))
    x = rng.uniform(0.0, 1.0, n)
    ax = np.array([va[rp[i]:rp[i + 1]] @ x[ci[rp[i]:rp[i + 1]]] for i in range(m)])
    lc, uc = ax - rng.uniform(0.0, 1.0, m), ax + rng.uniform(0.0, 1.0, m)
    kind = rng.integers(0, 3, m)
    uc[kind == 0] = np.inf
    lc[kind == 1] = uc[kind == 1] = ax[kind == 1]
    uv = rng.uniform(1.0, 3.0, n)
    uv[::3] = np.inf
    return dict(m=m, n=n, rowptr=rp, colidx=ci, val=va, c=rng.uniform(0.1, 1.0, n), lc=lc, uc=uc, lv=np.zeros(n), uv=uv)


def _ragged(parts):
    ms, ns, nz = ([p["m"] for p in parts], [p["n"] for p in parts], [len(p["val"]) for p in parts])
    ro, co, eo = (np.concatenate([[0], np.cumsum(v)]) for v in (ms, ns, nz))
    i32 = lambda a: np.asarray(a, dtype=np.int32)  # noqa: E731
    kw = {k: np.concatenate([p[k] for p in parts]) for k in ("val", *KEYS)}
    return dict(shared_a=False, batch=len(parts), m=int(ro[-1]), n=int(co[-1]), row_off=i32(ro), col_off=i32(co),
                rowptr=i32(np.concatenate([[0]] + [p["rowptr"][1:] + e for p, e in zip(parts, eo)])),
                colidx=i32(np.concatenate([p["colidx"] + c for p, c in zip(parts, co)])), **kw)


# 130 nonexpansive steps of rounding 70 x 1e-16 (the longest row) of the iterates'
# size, times the spread of the scaling (below 1e3)
TOL = 1e-9
# the norm estimate's setup sums in an order of its own for each batch: run it to
# rounding, or the step sizes differ by the 1e-7 at which it stops by default
OPTS = dict(eps=1e-13, iteration_limit=130, power_tol=1e-13)


def _check(got, want, what):
    assert np.abs(got - want).max(initial=0.0) <= TOL * (1.0 + np.abs(want).max(initial=0.0)), what


def _off_chip(parts, rng):
    """Results of parts from the memory-resident kernel."""
    from paper_2412_09734_amd.solver import BatchSolver
    wide = _instance(3, 8200, rng)
    with BatchSolver(**_ragged(parts + [wide]), **OPTS) as bs:
        x, y, res = bs.solve()
    return to_np(x), to_np(y), [res[b] for b in range(len(parts))]


# largest instance; one and two per thread at some of the thread counts, up to eight at the fewest
@pytest.mark.parametrize("m,n", [(60, 40), (33, 64), (120, 60), (64, 65), (250, 250), (120, 256), (130, 500), (500, 500),
                                 (513, 512), (500, 1000), (1000, 700), (900, 1500), (2048, 1100), (1500, 2049),
                                 (2100, 1000), (2500, 4096), (4096, 4096), (1000, 4097), (4200, 3600), (3500, 7000),
                                 (300, 8192), (3900, 8192)])
def test_columns_and_rows_per_thread(m, n):
    from paper_2412_09734_amd.solver import BatchSolver
    rng = np.random.default_rng(31 * m + n)
    parts = [_instance(mi, ni, rng) for mi, ni in [(m, n), (1, 1), (m // 2 + 1, n // 2 + 1), (0, 3), (m // 3, n // 4 + 1)]]
    need = max(m, n)
    x0, y0, r0 = _off_chip(parts, rng)
    kw = _ragged(parts)
    both = dict(parts[0], shared_a=True, batch=2, **{k: np.stack([parts[0][k]] * 2) for k in KEYS})
    # columns and rows per thread that a thread count gives, and what runs on chip:
    # two per thread always, up to eight while n + 3 m doubles and 3 KB fit 160 KB
    threads = [t for t in (64, 128, 256, 512, 1024)
               if need <= 2 * t or (need <= 8 * t and 8 * (n + 3 * m) + 3072 <= 160 * 1024)]
    assert threads
    _say(f"on chip, largest instance {m} x {n}, threads {threads} and the default")
    with BatchSolver(**kw, **OPTS) as bs, BatchSolver(**both, **OPTS) as sh:
        for t in [None] + threads:
            if t:
                bs.set_launch(t)
                sh.set_launch(t)
            x, y, res = bs.solve()
            _check(to_np(x), x0[:kw["n"]], (t, "x"))
            _check(to_np(y), y0[:kw["m"]], (t, "y"))
            xs, ys, rs = sh.solve()
            for b in range(2):
                _check(to_np(xs[b]), x0[:n], (t, "shared x"))
                _check(to_np(ys[b]), y0[:m], (t, "shared y"))
            for p, q in [(res[b], r0[b]) for b in range(len(parts))] + [(rs[0], r0[0]), (rs[1], r0[0])]:
                for f in ("status", "iterations", "restarts"):
                    assert p[f] == q[f], (t, f)


@pytest.mark.parametrize("m,n,threads", [(120, 100, 64), (60, 128, 64), (500, 260, 256), (256, 512, 256), (1500, 2048, 1024)])
def test_shared_matrix_with_short_slices(m, n, threads):
    """Two columns per thread on a shared matrix: rows and columns of at most 16
    entries stay in registers and LDS (longer ones are streamed, above)."""
    from paper_2412_09734_amd.solver import BatchSolver
    rng = np.random.default_rng(m + n)
    part = _instance(m, n, rng, longest=4)
    assert np.bincount(part["colidx"]).max() <= 16
    _say(f"short slices, shared {m} x {n}, {threads} threads")
    x0, y0, r0 = _off_chip([part], rng)
    both = dict(part, shared_a=True, batch=2, **{k: np.stack([part[k]] * 2) for k in KEYS})
    with BatchSolver(**both, **OPTS, threads=threads) as bs:
        x, y, res = bs.solve()
    for b in range(2):
        _check(to_np(x[b]), x0[:n], "x")
        _check(to_np(y[b]), y0[:m], "y")
        assert all(res[b][f] == r0[0][f] for f in ("status", "iterations", "restarts"))


@pytest.mark.parametrize("rays", [True, False])
@pytest.mark.parametrize("threads", [64, 128, None])
def test_statuses_and_certificates(oracle_lib, threads, rays):
    """Five and three columns per thread at 64 and 128 threads (streamed), one at
    the default: statuses and rays of the oracle."""
    from paper_2412_09734_amd.solver import BatchSolver
    _say(f"statuses at {threads or 'default'} threads, ray tests {'on' if rays else 'off'}")
    lps = [gen.infeasible_lp("duplicate_row", 150, 300, seed=5), gen.infeasible_lp("unbounded", 150, 300, seed=6),
           gen.planted_sparse_lp(150, 300, density=0.02, seed=7)]
    opts = dict(iteration_limit=20000 if rays else 1000)
    if not rays:
        opts.update(eps_primal_infeasible=0.0, eps_dual_infeasible=0.0)
    with BatchSolver.from_lps(lps, threads=threads, **opts) as bs:
        x, y, res = bs.solve()
        for b, lp in enumerate(lps):
            xo, yo, ro = oracle_lib.Oracle(lp, **opts).solve()
            cs, rs = bs.instance_slices(b)
            _say(b, res[b]["status_name"], res[b]["iterations"], ro["iterations"])
            assert res[b]["status"] == ro["status"] and res[b]["iterations"] == ro["iterations"]
            # certificates are differences of close points: 1e-6 as in the other batch tests
            got, want = (to_np(y[rs]), yo) if res[b]["status"] == 2 else (to_np(x[cs]), xo)
            assert rel_inf(got, want) <= 1e-6


@pytest.mark.parametrize("m,n", [(200, 8300), (8300, 300), (4700, 6000)])
def test_off_chip_at_the_default_launch(oracle_lib, m, n):
    """More than 8,192 columns (rows), or n + 3 m doubles beyond the LDS: the
    memory-resident kernel, 512 threads with the ray tests."""
    from paper_2412_09734_amd.solver import BatchSolver
    _say(f"off chip, {m} x {n}")
    lps = [gen.planted_sparse_lp(m, n, density=0.004, seed=3960), gen.ragged_planted_batch(1, 60, 60, seed=3961)[0]]
    with BatchSolver.from_lps(lps, iteration_limit=3000) as bs:
        x, y, res = bs.solve()
        for b, lp in enumerate(lps):
            xo, yo, ro = oracle_lib.Oracle(lp, iteration_limit=3000).solve()
            cs, rs = bs.instance_slices(b)
            assert res[b]["status"] == ro["status"] and res[b]["iterations"] == ro["iterations"], (b, res[b], ro)
            kb = oracle_lib.kkt(lp, to_np(x[cs]), to_np(y[rs]))
            assert abs(kb["kkt"] - res[b]["kkt_rel"]) <= 1e-9 + 1e-6 * kb["kkt"]
            assert rel_inf(to_np(x[cs]), xo) <= 1e-6
