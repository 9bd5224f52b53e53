"""The reverse pass over slices of 0 to 9 pairs (groups of four, two and one in
flight) and its batch sizes: instances whose rows and columns have every length
from 0 to 18 against the memory-resident kernel, which an instance of more than
8,192 columns and rows together sends all of them to. Tolerance 1e-9 as in the other
tests of the reverse pass."""

import sys

import numpy as np
import pytest

from gpu_util import to_np
from test_gpu_batch_stream import _instance, _ragged

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threads", [64, 256, 1024])
def test_reverse_pass(threads):
    from paper_2412_09734_amd.solver import BatchSolver
    print(f"case: reverse pass, {threads} threads", file=sys.stderr, flush=True)
    rng = np.random.default_rng(5)
    parts = []
    for k in range(19):                       # one slice of rows of length k each
        p = _instance(64, 70, rng, longest=0)
        cols = [np.sort(rng.choice(70, k, replace=False)) for _ in range(64)]
        p.update(rowptr=np.arange(65) * k, colidx=np.concatenate(cols), val=rng.standard_normal(64 * k),
                 uc=np.full(64, np.inf), lc=rng.uniform(-1.0, 0.0, 64))
        parts.append(p)
    wide = _instance(3, 8200, rng)
    T = 70
    kw, ref = _ragged(parts), _ragged(parts + [wide])
    gx, gy = rng.standard_normal(ref["n"]), rng.standard_normal(ref["m"])
    out = []
    for q in (kw, ref):
        with BatchSolver(**q, threads=threads) as bs:
            bs.unrolled(T)
            out.append([to_np(v) for v in bs.backward(gx[:q["n"]], gy[:q["m"]])])
    for u, v in zip(*out):
        v = v[:len(u)]
        assert np.abs(u - v).max() <= 1e-9 * (1.0 + np.abs(v).max())
