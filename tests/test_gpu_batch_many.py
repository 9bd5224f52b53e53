"""Ragged batches at the ends of the slice order: more instances than a launch of
one workgroup each can hold, and instances of thousands of rows
with many equal lengths."""

import sys

import numpy as np
import pytest

from gpu_util import to_np

pytestmark = pytest.mark.gpu


# workgroups of 1,024 and of 256 threads
@pytest.mark.parametrize("B", [(1 << 22) + 5, (1 << 24) + 5])
def test_more_instances_than_a_launch_holds(B):
    """min x s.t. x = b (even instances) or x >= b (odd ones), 0 <= x <= 2."""
    import torch
    from paper_2412_09734_amd.solver import BatchSolver
    print(f"case: {B} instances of one row and one column", file=sys.stderr, flush=True)
    d = dict(dtype=torch.float64, device="cuda")
    off = torch.arange(B + 1, dtype=torch.int32, device="cuda")
    one, zero = torch.ones(B, **d), torch.zeros(B, **d)
    b = (torch.arange(B, **d) % 7 + 1.0) / 8.0
    uc = b.clone()
    uc[1::2] = float("inf")
    with BatchSolver(shared_a=False, batch=B, m=B, n=B, rowptr=off, colidx=off[:B], val=one, c=one, lc=b, uc=uc,
                     lv=zero, uv=2.0 * one, row_off=off.cpu(), col_off=off.cpu(), power_max_iters=4, eps=1e-9) as bs:
        x, y, res = bs.solve()
    # the relative KKT error is at most 1e-9 on entries of size 1
    assert float((x - b).abs().max()) <= 1e-8 and float((y - 1.0).abs().max()) <= 1e-8
    for k in (0, 1, (1 << 22) - 1, 1 << 22, B - 1):
        assert res[k]["status_name"] == "optimal", (k, res[k])


def _csr(lens, n, rng):
    cols = [np.sort(rng.choice(n, k, replace=False)) for k in lens]
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), np.concatenate(cols).astype(np.int32)


@pytest.mark.parametrize("m,n", [(1, 1), (63, 64), (65, 129), (1023, 2049), (4097, 300), (8192, 40)])
def test_order_of_unequal_rows(m, n):
    """The middle one of three instances solved alone on a shared matrix, whose
    rows keep their order, takes the same steps. Tolerance: 65 nonexpansive steps
    of rounding 40 x 1e-16 of the iterates' size, times the spread of the scaling
    (below 1e3)."""
    from paper_2412_09734_amd.solver import BatchSolver
    print(f"case: ragged order of {m} x {n}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(m + n)
    lens = np.minimum(rng.integers(0, 40, m) // rng.integers(1, 9, m), n)
    lens[m // 2] = min(n, 70)
    rp, ci = _csr(lens, n, rng)
    va = rng.standard_normal(len(ci))
    x0 = rng.uniform(0.0, 1.0, n)
    ax = np.add.reduceat(np.append(va * x0[ci], 0.0), rp[:-1]) * (lens > 0)
    one = dict(rowptr=rp, colidx=ci, val=va, c=rng.uniform(0.1, 1.0, n), lc=ax - 0.1, uc=ax + 0.2, lv=np.zeros(n),
               uv=np.full(n, 2.0))
    opts = dict(eps=1e-13, iteration_limit=65)
    with BatchSolver(shared_a=True, batch=1, m=m, n=n, **one, **opts) as bs:
        xs, ys, _ = bs.solve()
    three = {k: np.concatenate([one[k]] * 3) for k in ("val", "c", "lc", "uc", "lv", "uv")}
    three["rowptr"] = np.concatenate([[0]] + [rp[1:] + k * rp[-1] for k in range(3)]).astype(np.int32)
    three["colidx"] = np.concatenate([ci + k * n for k in range(3)]).astype(np.int32)
    with BatchSolver(shared_a=False, batch=3, m=3 * m, n=3 * n, row_off=np.arange(4) * m, col_off=np.arange(4) * n,
                     **three, **opts) as bs:
        x, y, _ = bs.solve()
    for got, want, k in ((to_np(x), to_np(xs).reshape(-1), n), (to_np(y), to_np(ys).reshape(-1), m)):
        for b in range(3):
            assert np.abs(got[b * k:(b + 1) * k] - want).max() <= 1e-9 * (1.0 + np.abs(want).max())
