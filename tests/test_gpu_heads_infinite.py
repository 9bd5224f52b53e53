"""Infinite decisions in the QP value: factor columns that only pad the rank to
whole groups of eight add nothing, not NaN."""

import sys

import numpy as np
import pytest

from gpu_util import to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r", [(3, 0), (70, 1), (300, 5), (300, 8), (40, 20), (257, 31)])
def test_qp_value_of_an_infinite_point(n, r):
    import torch
    from paper_2412_09734_amd import heads as h
    print(f"case: QP value, infinite x, n={n} r={r}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(n + r)
    F, d, c = rng.uniform(0.1, 1.0, (n, r)), rng.uniform(0.1, 1.0, (2, n)), rng.uniform(0.0, 1.0, (2, n))
    x = rng.uniform(0.1, 1.0, (2, n))
    x[0, n // 2] = np.inf
    Fa = F if r else torch.empty(n, 0, dtype=torch.float64)
    value, gx = (to_np(t) for t in h.qp_value(Fa, d, c, x))
    with np.errstate(invalid="ignore"):
        want = (x @ F) @ F.T + d * x + c
    assert value[0] == np.inf and np.isfinite(value[1])
    assert np.array_equal(np.isinf(gx), np.isinf(want)) and not np.isnan(gx).any()
    if r:
        assert np.isinf(gx[0]).all()
