"""The layer's products with sliced rows against plain ones (CPU, float64):
values, gradients and their layout, rows divisible and not, frozen weights."""
import pytest
import torch

from paper_2604_03815_amd.layer import _matmul_rows


@pytest.mark.parametrize("n", [1, 255, 1024, 1025, 1031, 4099, 17226])
@pytest.mark.parametrize("frozen", [False, True])
def test_sliced_products(n, frozen):
    g = torch.Generator().manual_seed(n)
    x = torch.randn(n, 12, generator=g, dtype=torch.float64, requires_grad=True)
    ws = [torch.randn(12, m, generator=g, dtype=torch.float64, requires_grad=not (frozen and m == 5)) for m in (3, 5, 8)]
    leaves = [x] + [w for w in ws if w.requires_grad]
    plain, sliced = [x @ w for w in ws], _matmul_rows(x, ws)
    go = [torch.randn(t.shape, generator=g, dtype=torch.float64) for t in plain]
    for a, b in zip(plain, sliced):
        torch.testing.assert_close(b, a, rtol=1e-12, atol=1e-12)
    # sums of n products in another order: n 2^-53 times a few
    for a, b in zip(torch.autograd.grad(plain, leaves, go), torch.autograd.grad(sliced, leaves, go)):
        torch.testing.assert_close(b, a, rtol=1e-10, atol=1e-10)
        assert b.is_contiguous()
    with torch.no_grad():
        for a, b in zip(plain, _matmul_rows(x, ws)):
            assert torch.equal(a, b)
