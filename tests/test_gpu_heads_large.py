"""Loss heads on many small samples, rows or instances: calls whose arrays fit
the card, up to the 2^32 work-items that one launch can hold, and the entry
arithmetic of the kernels at the edges of their tiles. Entries that are formed
one by one are compared exactly."""

import sys

import numpy as np
import pytest

from gpu_util import to_np

pytestmark = pytest.mark.gpu


def _say(*a):
    print("case:", *a, file=sys.stderr, flush=True)


@pytest.mark.parametrize("B,M,n", [(1, 1, 1), (5, 9, 1), (1, 5000, 2), (300, 1, 7), (7, 3, 341), (2, 3, 511),
                                   (2, 3, 512), (1, 4, 513), (3, 2, 1023), (40, 100, 24)])
def test_perturbed_costs_tiles(B, M, n):
    from paper_2412_09734_amd import heads as h
    _say(f"perturbed costs B={B} M={M} n={n}")
    rng = np.random.default_rng(B + M + n)
    ch, Z = rng.standard_normal((B, n)), rng.standard_normal((B, M, n))
    assert np.array_equal(to_np(h.pfy_costs(ch, Z, 0.3)), ch[:, None] + 0.3 * Z)


@pytest.mark.parametrize("n,M,p", [(255, 2, 4), (257, 5, 5), (512, 7, 8), (513, 8, 9), (768, 9, 16), (1023, 11, 1),
                                   (2048, 13, 3), (2049, 1, 17), (4097, 3, 2), (6145, 15, 24)])
def test_groups_of_loads(n, M, p):
    """Columns, samples and features around the groups whose loads are in flight
    together: small whole numbers, so that every sum is exact in any order."""
    from paper_2412_09734_amd import heads as h
    _say(f"groups of loads n={n} M={M} p={p}")
    rng = np.random.default_rng(n)
    i = lambda *s: rng.integers(-8, 9, s).astype(float)  # noqa: E731
    B = 3
    x, c, w, s, z = i(B, n), i(B, n), i(B, n), i(B, n), i(B)
    assert np.array_equal(to_np(h.regret(c, x, z)), (c * x).sum(1) - z)
    loss, grad = h.spo_plus(x, c, w, z, s)
    assert np.array_equal(to_np(loss), (2 * x * (w - s) + c * s).sum(1) - z)
    assert np.array_equal(to_np(grad), 2 * (w - s))
    Z, wm = i(B, M, n), M * i(B, M, n)
    loss, grad = h.pfy(c, w, Z, 2.0, wm)
    assert np.array_equal(to_np(loss), (c * w).sum(1) - ((c[:, None] + 2 * Z) * wm).sum((1, 2)) / M)
    assert np.array_equal(to_np(grad), w - wm.sum(1) / M)
    f, W = i(B, n, p), i(p)
    assert np.array_equal(to_np(h.linear_costs(f, W)), f @ W)
    assert np.array_equal(to_np(h.linear_costs_backward(f, x)), (f * x[..., None]).sum((0, 1)))


@pytest.mark.parametrize("B,M,n", [(1, (1 << 24) + 3, 1), ((1 << 24) + 5, 1, 2), (1 << 13, 1 << 12, 3)])
def test_perturbed_costs_of_many_samples(B, M, n):
    import torch
    from paper_2412_09734_amd import heads as h
    _say(f"perturbed costs of {B} x {M} samples, n={n}")
    g = torch.Generator(device="cuda").manual_seed(n)
    ch = torch.rand(B, n, dtype=torch.float64, device="cuda", generator=g)
    Z = torch.rand(B, M, n, dtype=torch.float64, device="cuda", generator=g)
    want = 0.5 * Z
    want += ch[:, None]
    assert torch.equal(h.pfy_costs(ch, Z, 0.5), want)


@pytest.mark.parametrize("B,M,n", [(5, 1 << 20, 820), (1, 3, 1431655771), (1, (1 << 31) - 1, 3)])
def test_perturbed_costs_past_32_bits(B, M, n):
    """2^32 entries and more: several launches, of instances or of one's samples."""
    import torch
    from paper_2412_09734_amd import heads as h
    _say(f"perturbed costs of {B * M * n} entries, n={n}")
    ch = torch.arange(1.0, B * n + 1, dtype=torch.float64, device="cuda").view(B, n) % 1009.0
    Z = torch.zeros(B, M, n, dtype=torch.float64, device="cuda")
    flat = Z.view(-1)
    N = B * M * n
    at = torch.tensor([0, 511, (1 << 32) // n * n - 1, (1 << 32) // n * n, (1 << 32) - 1, 1 << 32, N - 1], device="cuda")
    at = at[at < N]
    flat[at] = 8.0
    out = h.pfy_costs(ch, Z, 0.5)
    # every entry, by blocks of samples: whole numbers, exact
    step = max(1, (1 << 28) // n)
    for b in range(B):
        for m in range(0, M, step):
            Z[b, m:m + step].mul_(0.5).add_(ch[b])
    assert torch.equal(out, Z)


@pytest.mark.parametrize("rows,p", [((1 << 28) + 5, 17), ((1 << 32) + 5, 1)])
def test_costs_of_many_rows(rows, p):
    """Features that are zero but for the first, the last and a few other rows."""
    import torch
    from paper_2412_09734_amd import heads as h
    _say(f"cost model on {rows} rows of {p} features")
    B = 3
    assert rows % B == 0
    f = torch.zeros(B, rows // B, p, dtype=torch.float64, device="cuda")
    flat = f.view(-1, p)
    at = torch.tensor([0, 1, 255, 256, 4096, (1 << 28) - 1, rows // 2, rows - 2, rows - 1], device="cuda")
    flat[at] = torch.arange(1.0, at.numel() * p + 1, dtype=torch.float64, device="cuda").view(-1, p)
    W = torch.arange(1.0, p + 1, dtype=torch.float64, device="cuda")
    c = h.linear_costs(f, W).view(-1)
    # whole numbers: the sums are exact in any order
    assert torch.equal(c[at], (flat[at] * W).sum(1))
    assert int(torch.count_nonzero(c)) == at.numel()


def test_spo_costs_of_many_entries():
    import torch
    from paper_2412_09734_amd import heads as h
    B, n = 3, ((1 << 32) + 2) // 3
    _say(f"SPO+ costs of {B} x {n} entries")
    c = torch.zeros(B, n, dtype=torch.float64, device="cuda")
    flat = c.view(-1)
    at = torch.tensor([0, 1, 256, (1 << 31) + 1, B * n - 300, B * n - 1], device="cuda")
    flat[at] = torch.arange(1.0, 7.0, dtype=torch.float64, device="cuda")
    out = h.spo_plus_costs(c, c).view(-1)
    assert torch.equal(out[at], flat[at])
    assert int(torch.count_nonzero(out)) == at.numel()


@pytest.mark.parametrize("B,n", [((1 << 22) + 3, 1025), ((1 << 24) + 3, 1)])
def test_losses_of_many_instances(B, n):
    """One buffer of small whole numbers in every role: all sums are exact."""
    import torch
    from paper_2412_09734_amd import heads as h
    _say(f"regret, SPO+, Fenchel-Young and QP value of {B} instances, n={n}")
    x = torch.zeros(B, n, dtype=torch.float64, device="cuda")
    at = torch.tensor([0, 1, (1 << 21) - 1, 1 << 21, (1 << 22) - 1, B - 2, B - 1], device="cuda")
    x[at] = torch.arange(1.0, at.numel() * n + 1, dtype=torch.float64, device="cuda").view(-1, n) % 64
    vs = torch.ones(B, dtype=torch.float64, device="cuda")
    want = torch.zeros(B, dtype=torch.float64, device="cuda")
    want[at] = (x[at] ** 2).sum(1)
    assert torch.equal(h.regret(x, x, vs), want - 1.0)
    loss, grad = h.spo_plus(x, x, x, vs, x)
    assert torch.equal(loss, want - 1.0) and int(torch.count_nonzero(grad)) == 0
    del grad
    loss, grad = h.pfy(x, x, x.view(B, 1, n), 1.0, x.view(B, 1, n))
    assert torch.equal(loss, -want) and int(torch.count_nonzero(grad)) == 0
    del grad
    value, gx = h.qp_value(torch.zeros(n, 0, dtype=torch.float64, device="cuda"), x, x, x)
    want[at] = (x[at] ** 2 + 0.5 * x[at] ** 3).sum(1)
    assert torch.equal(value, want)
    assert torch.equal(gx[at], x[at] ** 2 + x[at])
