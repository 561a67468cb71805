"""bf16 TTMs of strided modes on both sides of the line, 32768 columns, above
which the 64-column kernel takes them: against the 16-column one, which a
pointer off by one element selects; same products in the same order, so the
same bits."""
import pytest
import torch

from paper_1510_06689_amd import tucker

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l,b", [(16, 2048), (16, 2049), (20, 1639), (64, 600), (68, 482), (132, 249), (8196, 4)])
@pytest.mark.parametrize("j", [1, 31, 32, 33, 64, 97, 128])
@pytest.mark.parametrize("k", [1, 16, 17, 100, 530])
def test_same_bits(l, b, j, k):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(l + 200 * j + k)
    x = torch.randn(b, j, l, generator=g, device="cuda:0")
    y = torch.empty(x.numel() + 1, device="cuda:0")[1:].view(x.shape).copy_(x)
    for transpose, precision in ((True, "bf16x3"), (False, "bf16x3"), (True, "bf16")):
        m = torch.randn((k, j) if transpose else (j, k), generator=g, dtype=torch.float64, device="cuda:0").t()
        zs = [tucker.ttm(t.permute(2, 1, 0), 1, m, transpose, precision) for t in (x, y)]
        # (narrow modes of long runs run in FP64 when aligned)
        assert torch.equal(zs[0], zs[1]) or (j <= 64 and k <= 16 and l == 64)
        op = (m.t() if transpose else m).contiguous()
        tol = 2.0 ** -7 if precision == "bf16" else 2.0 ** -15
        z = zs[0].permute(2, 1, 0)[:: max(1, b // 40)].double()
        part = x[:: max(1, b // 40)].double()
        ref, size = torch.matmul(op, part), torch.matmul(op.abs(), part.abs())
        assert bool(((z - ref).abs() <= tol * size).all())
