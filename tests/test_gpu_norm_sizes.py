"""The norm estimate of one problem at the sizes where a half step's vector work
changes hands: blocks of 256, 1,024 threads, 8 elements a thread (one launch up
to 8,192 elements, three beyond), against the CPU oracle."""

import sys

import pytest

from test_gpu_batch_norm import _path

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nodes", [40, 256, 257, 1024, 1026, 2049, 8192, 8193, 8194])
def test_norm_sizes(oracle_lib, nodes):
    from paper_2412_09734_amd.solver import Solver
    print(f"case: norm estimate, path of {nodes} nodes", file=sys.stderr, flush=True)
    lp = _path(nodes)
    opts = dict(power_max_iters=40, power_tol=1e-12, iteration_limit=2)
    with Solver.from_lp(lp, **opts) as s:
        r = s.solve()[2]
    sc = oracle_lib.Oracle(lp, **opts).scaling()
    assert abs(r["eta"] - sc["eta"]) <= 1e-10 * sc["eta"]
    assert abs(r["power_iters"] - sc["power_iters"]) <= (0 if sc["power_iters"] == 40 else 1)
