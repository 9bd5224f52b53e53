"""The batched solve that keeps a narrow shared matrix in registers, at the edges
of its shapes (columns and rows per thread, wave remainders, empty rows and
columns) and of its momentum table, against the general kernels at 128 threads."""

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
@pytest.mark.parametrize("m,n", [(1, 1), (3, 2), (64, 128), (255, 511), (256, 512), (256, 513), (250, 1000),
                                 (256, 1024), (257, 1024), (300, 1025), (512, 2047), (513, 2048), (700, 2500),
                                 (1024, 4095), (1024, 4096)])
@pytest.mark.parametrize("check_every,limit", [(1, 9), (64, 150), (100, 250)])
def test_resident_solve(m, n, check_every, limit):
    from paper_2412_09734_amd.solver import BatchSolver
    print(f"case: resident matrix {m} x {n}, check every {check_every}", file=sys.stderr, flush=True)
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
    kw = dict(shared_a=True, batch=B, m=m, n=n, rowptr=rowptr, colidx=np.nonzero(nz)[1].astype(np.int32),
              val=a[nz], c=rng.uniform(0.1, 1.0, (B, n)), lc=lc, uc=uc, lv=lv, uv=uv)
    with BatchSolver(**kw, eps=1e-13, check_every=check_every, iteration_limit=limit) as bs:
        runs = {}
        for threads in (128, 256, 512):
            bs.set_launch(threads)
            runs[threads] = bs.solve()
    x0, y0, r0 = runs[128]
    # at most 250 nonexpansive steps of rounding 1e-16 of the iterates' size,
    # times the spread of the scaling: 1e-10 leaves a factor 1,000
    for threads in (256, 512):
        x, y, r = runs[threads]
        for b in range(B):
            assert r[b]["status"] == r0[b]["status"] and r[b]["iterations"] == r0[b]["iterations"]
            assert r[b]["restarts"] == r0[b]["restarts"]
            for u, v in ((x[b], x0[b]), (y[b], y0[b])):
                u, v = to_np(u), to_np(v)
                assert np.abs(u - v).max(initial=0.0) <= 1e-10 * (1.0 + np.abs(v).max(initial=0.0))
            for key in ("primal_obj", "dual_obj"):
                assert abs(r[b][key] - r0[b][key]) <= 1e-9 * (1.0 + abs(r0[b][key]))
