"""The batched solve that keeps a narrow shared matrix in registers, at the edges
of its shapes (columns and rows per thread, wave remainders, empty rows and
columns) and of its momentum table, and its unrolled forward and reverse passes,
against the general kernels at 128 threads."""

import sys

import numpy as np
import pytest

from gpu_util import to_np

pytestmark = pytest.mark.gpu


def _narrow(m, n, rng):
    """At most 2 entries a column and 8 a row; the last row and column are empty if there is room."""
    slots = rng.permutation(np.repeat(np.arange(m if m < 3 or 8 * (m - 1) < 2 * n else m - 1), 8))[:2 * n]
    a = np.zeros((m, n))
    for j in range(min(n, len(slots) // 2)):
        for i in slots[2 * j:2 * j + 2]:
            a[i, j] = rng.choice([-1.0, 1.0]) * rng.uniform(0.5, 2.0)
    if n > 2:
        a[:, n - 1] = 0.0
    return a


# (m, n): 2, 4 and 8 columns a thread at 256 and 512 threads, each with a remainder
SHAPES = [(1, 1), (3, 2), (64, 128), (255, 511), (256, 512), (256, 513), (250, 1000), (256, 1024), (257, 1024),
          (300, 1025), (512, 2047), (513, 2048), (700, 2500), (1024, 4095), (1024, 4096)]


def _batch(m, n):
    rng = np.random.default_rng(7 * m + n)
    a = _narrow(m, n, rng)
    B = 3
    xs = rng.uniform(0.0, 1.0, (B, n))
    ax = xs @ a.T
    lc, uc = ax - rng.uniform(0.0, 1.0, (B, m)), ax + rng.uniform(0.0, 1.0, (B, m))
    kind = rng.integers(0, 4, m)
    lc[:, kind == 1] = uc[:, kind == 1] = ax[:, kind == 1]
    lc[:, kind == 2] = -np.inf
    uc[:, kind == 3] = np.inf
    lv, uv = np.zeros((B, n)), rng.uniform(1.0, 3.0, (B, n))
    uv[:, ::3] = np.inf
    lv[:, 1::5] = -4.0
    nz = a != 0
    rowptr = np.concatenate([[0], np.cumsum(nz.sum(1))]).astype(np.int32)
    return dict(shared_a=True, batch=B, m=m, n=n, rowptr=rowptr, colidx=np.nonzero(nz)[1].astype(np.int32),
                val=a[nz], c=rng.uniform(0.1, 1.0, (B, n)), lc=lc, uc=uc, lv=lv, uv=uv)


def _near(u, v):
    u, v = to_np(u), to_np(v)
    return np.abs(u - v).max(initial=0.0) <= 1e-10 * (1.0 + np.abs(v).max(initial=0.0))


# at most 250 nonexpansive steps of rounding 1e-16 of the iterates' size, times
# the spread of the scaling: the bound of 1e-10 leaves a factor 1,000
@pytest.mark.parametrize("m,n", SHAPES)
@pytest.mark.parametrize("check_every,limit", [(1, 9), (64, 150), (100, 250)])
def test_resident_solve(m, n, check_every, limit):
    from paper_2412_09734_amd.solver import BatchSolver
    print(f"case: resident matrix {m} x {n}, check every {check_every}", file=sys.stderr, flush=True)
    kw = _batch(m, n)
    with BatchSolver(**kw, eps=1e-13, check_every=check_every, iteration_limit=limit) as bs:
        runs = {}
        for threads in (128, 256, 512):
            bs.set_launch(threads)
            runs[threads] = bs.solve()
    x0, y0, r0 = runs[128]
    for threads in (256, 512):
        x, y, r = runs[threads]
        for b in range(kw["batch"]):
            assert r[b]["status"] == r0[b]["status"] and r[b]["iterations"] == r0[b]["iterations"]
            assert r[b]["restarts"] == r0[b]["restarts"]
            assert _near(x[b], x0[b]) and _near(y[b], y0[b])
            for key in ("primal_obj", "dual_obj"):
                assert abs(r[b][key] - r0[b][key]) <= 1e-9 * (1.0 + abs(r0[b][key]))


# the reverse pass is linear in the cotangents with the same factors, so the
# same bound holds for it
@pytest.mark.parametrize("m,n", SHAPES)
@pytest.mark.parametrize("check_every,T", [(64, 1), (1, 9), (64, 65), (64, 131), (100, 230)])
def test_resident_unrolled(m, n, check_every, T):
    from paper_2412_09734_amd.solver import BatchSolver
    print(f"case: resident matrix {m} x {n}, {T} unrolled iterations", file=sys.stderr, flush=True)
    kw = _batch(m, n)
    rng = np.random.default_rng(T)
    gx, gy = rng.standard_normal((kw["batch"], n)), rng.standard_normal((kw["batch"], m))
    with BatchSolver(**kw, check_every=check_every) as bs:
        runs = {}
        for threads in (128, 256, 512):
            bs.set_launch(threads)
            out = bs.unrolled(T)
            again = bs.unrolled(T, replay=True)
            assert np.array_equal(to_np(out[0]), to_np(again[0])) and np.array_equal(to_np(out[1]), to_np(again[1]))
            runs[threads] = (*out, *bs.backward(gx, gy))
    for threads in (256, 512):
        assert len(runs[threads]) == len(runs[128])
        for u, v in zip(runs[threads], runs[128]):
            assert _near(u, v)
