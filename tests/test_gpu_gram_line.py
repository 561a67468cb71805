"""FP64 Gram on both sides of the line, 4096 columns, up to which small tensors
take schedules of their own (tiles of 32 columns up to 64 rows, pair groups
over many workgroups above 160): contiguous, packed and strided columns, the
edges of a tile and of the block counts, both storage types."""
import pytest
import torch

from paper_1510_06689_amd import tucker

pytestmark = pytest.mark.gpu
U = 2.0 ** -53

EXTENTS = [1, 8, 16, 17, 32, 33, 48, 49, 64, 65, 96, 113, 128, 144, 160, 161, 176, 192, 193, 224, 225, 256, 257, 320, 321, 384, 400, 512]


def _check(l, j, b, dtype):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(l + 7 * j + b)
    x = torch.randn(b, j, l, generator=g, dtype=torch.float64, device="cuda:0").to(dtype)
    s, nu = tucker.gram(x.permute(2, 1, 0), 1)
    a = x.double().permute(1, 0, 2).reshape(j, -1)
    ref = a @ a.t()
    # K products and sums on either side, each rounded: at most K u |a_i||a_j|
    d = ref.diagonal().sqrt()
    assert bool(((s - ref).abs() <= 2 * a.shape[1] * U * d[:, None] * d[None, :]).all())
    assert torch.equal(s, s.t())
    assert abs(float(nu) - float(ref.trace())) <= 2 * (a.shape[1] + j) * U * float(ref.trace())


@pytest.mark.parametrize("j", EXTENTS)
def test_few_columns(j):
    for l, b in [(1, 1), (1, 15), (1, 17), (1, 530), (1, 4096), (3, 5), (3, 1365), (15, 11), (16, 256), (17, 240), (31, 132), (33, 124), (100, 40), (4096, 1)]:
        _check(l, j, b, torch.float64 if (l + b) % 2 else torch.float32)


@pytest.mark.parametrize("j", EXTENTS)
def test_more_columns(j):
    for l, b in [(1, 4097), (3, 1501), (20, 431), (65, 64), (129, 33), (4100, 1)]:
        _check(l, j, b, torch.float64 if (l + b) % 2 else torch.float32)
