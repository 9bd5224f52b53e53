"""The loss heads at the edges of their kernels (feature counts around the two
cost-model variants, instances around the workgroup sizes, single entries)
against numpy; sums within 1e-14 per added term of the absolute terms, products
that are formed one by one exactly."""

import sys

import numpy as np
import pytest

from gpu_util import to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,n,p", [(1, 1, 1), (2, 255, 3), (1, 257, 8), (3, 700, 15), (3, 700, 16), (3, 700, 17),
                                   (2, 513, 33), (5, 1031, 63), (4, 300, 64), (70, 1024, 5), (40, 1025, 7)])
def test_cost_model_shapes(B, n, p):
    from paper_2412_09734_amd import heads as h
    print(f"case: cost model heads B={B} n={n} p={p}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(n + p)
    f, W, gc = rng.standard_normal((B, n, p)), rng.standard_normal(p), rng.standard_normal((B, n))
    ct, x, vs = rng.standard_normal((B, n)), rng.standard_normal((B, n)), rng.standard_normal(B)
    assert np.all(np.abs(to_np(h.linear_costs(f, W)) - f @ W) <= 1e-14 * p * (np.abs(f) @ np.abs(W)) + 1e-300)
    assert np.all(np.abs(to_np(h.regret(ct, x, vs)) - ((ct * x).sum(1) - vs))
                  <= 1e-14 * n * ((np.abs(ct * x)).sum(1) + np.abs(vs)))
    want, scale = np.einsum("bn,bnp->p", gc, f), np.einsum("bn,bnp->p", np.abs(gc), np.abs(f))
    got = to_np(h.linear_costs_backward(f, gc))
    assert np.all(np.abs(got - want) <= 1e-14 * n * scale)
    import torch
    same = torch.empty(p, dtype=torch.float64, device="cuda")
    assert np.array_equal(to_np(h.linear_costs_backward_noalloc(f, gc, same)), got)


@pytest.mark.parametrize("B,n,M", [(1, 1, 1), (2, 63, 3), (2, 1024, 4), (2, 1025, 5), (3, 4099, 2)])
def test_surrogate_shapes(B, n, M):
    from paper_2412_09734_amd import heads as h
    print(f"case: surrogate heads B={B} n={n} M={M}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(n)
    ch, ct, ws, wt = (rng.standard_normal((B, n)) for _ in range(4))
    zs, Z, wm = rng.standard_normal(B), rng.standard_normal((B, M, n)), rng.standard_normal((B, M, n))
    loss, grad = h.spo_plus(ch, ct, ws, zs, wt)
    assert np.array_equal(to_np(grad), 2.0 * (ws - wt))
    terms = np.abs(2 * ch * (ws - wt)) + np.abs(ct * wt)
    assert np.all(np.abs(to_np(loss) - ((2 * ch * (ws - wt) + ct * wt).sum(1) - zs)) <= 1e-14 * n * (terms.sum(1) + np.abs(zs)))
    cp = ch[:, None] + 0.3 * Z
    assert np.array_equal(to_np(h.pfy_costs(ch, Z, 0.3)), cp)
    loss, grad = h.pfy(ch, ws, Z, 0.3, wm)
    assert np.all(np.abs(to_np(grad) - (ws - wm.mean(1))) <= 1e-14 * M * (np.abs(ws) + np.abs(wm).sum(1)))
    terms = np.abs(ch * ws) + np.abs(cp * wm).sum(1)
    assert np.all(np.abs(to_np(loss) - ((ch * ws).sum(1) - (cp * wm).sum(2).mean(1))) <= 1e-14 * n * M * terms.sum(1))


@pytest.mark.parametrize("B,n,r", [(1, 1, 1), (2, 255, 8), (2, 257, 9), (3, 500, 20), (2, 300, 32), (2, 70, 0)])
def test_qp_value_shapes(B, n, r):
    import torch
    from paper_2412_09734_amd import heads as h
    print(f"case: QP value B={B} n={n} r={r}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(n + r)
    F, d, c, x = rng.standard_normal((n, r)), rng.random((B, n)), rng.standard_normal((B, n)), rng.standard_normal((B, n))
    Fa = F if r else torch.empty(n, 0, dtype=torch.float64)
    value, gx = h.qp_value(Fa, d, c, x)
    qx = (x @ F) @ F.T + d * x
    scale = (np.abs(x) @ np.abs(F)) @ np.abs(F).T + np.abs(d * x) + np.abs(c)
    assert np.all(np.abs(to_np(gx) - (qx + c)) <= 1e-14 * (n + r) * scale)
    assert np.all(np.abs(to_np(value) - (x * (0.5 * qx + c)).sum(1)) <= 1e-14 * n * (n + r) * (np.abs(x) * scale).sum(1))
