"""The tiled GEMM at K that is no multiple of its K slab (128 values): the
slab's exponents come by one unaligned load per row, moved back to the row's
end for the last slab, and by single bytes in rows shorter than a slab."""
import pytest
import torch

import paper_2110_15456_amd as fb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("g", [16, 32])
@pytest.mark.parametrize("ma,mb", [(2, 4), (4, 2), (4, 4), (2, 2), (6, 6), (6, 4), (8, 8)])
@pytest.mark.parametrize("groups", [1, 3, 4, 5, 7, 8, 9, 15, 17, 31, 33, 259])
def test_ragged_k(groups, ma, mb, g):
    M, N, K = 65, 70, groups * g
    gen = torch.Generator(device="cuda").manual_seed(groups)
    # a different scale per row, so that another row's exponent shows
    a = torch.randn((M, K), device="cuda", generator=gen) * torch.logspace(-3, 3, M, device="cuda")[:, None]
    b = torch.randn((N, K), device="cuda", generator=gen) * torch.logspace(3, -3, N, device="cuda")[:, None]
    A, B = fb.quantize(a, g=g, m=ma), fb.quantize(b, g=g, m=mb)
    C = fb.gemm(A, B, workspace=False).double().cpu()
    x, y = fb.dequantize(A).double().cpu(), fb.dequantize(B).double().cpu()
    # at most one rounding per group and chunk pair of a sum bounded by sum |x| |y|
    bound = (4 * groups + 4) * 2.0**-24 * (x.abs() @ y.abs().T)
    assert bool(((C - x @ y.T).abs() <= bound).all())
