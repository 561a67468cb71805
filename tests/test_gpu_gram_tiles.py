"""FP64 Gram at the edges of its tiles: block counts with schedules of their
own, one and several tiles per workgroup, contiguous, packed and strided
columns, partial last tiles, both storage types."""
import pytest
import torch

from paper_1510_06689_amd import tucker

pytestmark = pytest.mark.gpu
U = 2.0 ** -53

EXTENTS = [1, 2, 15, 16, 17, 32, 33, 48, 49, 65, 81, 97, 113, 128, 129, 145, 177, 200, 225, 256, 257, 321, 385, 449, 512]


def _check(dims, mode, dtype):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(1 + mode + 7 * dims[mode])
    x = torch.randn(tuple(reversed(dims)), generator=g, dtype=torch.float64, device="cuda:0")
    x = x.to(dtype).permute(*reversed(range(len(dims))))
    s, nu = tucker.gram(x, mode)
    a = x.movedim(mode, 0).reshape(dims[mode], -1).double()
    ref = a @ a.t()
    # K products and sums on either side, each rounded: at most K u |a_i||a_j|
    d = ref.diagonal().sqrt()
    tol = 2 * a.shape[1] * U * d[:, None] * d[None, :]
    assert bool(((s - ref).abs() <= tol).all())
    assert torch.equal(s, s.t())
    assert abs(float(nu) - float(ref.trace())) <= 2 * (a.shape[1] + dims[mode]) * U * float(ref.trace())


@pytest.mark.parametrize("j", EXTENTS)
def test_contiguous(j):
    for cols in (1, 31, 33, 700):          # less than a tile, its edges, several
        _check((j, cols), 0, torch.float64)
    _check((j, 70001 if j < 200 else 9001), 0, torch.float32)   # several tiles per workgroup, odd count


@pytest.mark.parametrize("j", EXTENTS)
def test_packed_and_strided(j):
    _check((3, j, 301), 1, torch.float64)      # packed, a partial last tile, padding columns
    _check((10, j, 1), 1, torch.float32)       # one b-block
    _check((129, j, 5), 1, torch.float64)      # strided, segments of a partial width
    _check((7, 39, j, 23), 2, torch.float32)   # strided, L = 273


def test_many_tiles_per_workgroup():
    _check((128, 300007), 0, torch.float32)
    _check((33, 100, 2111), 1, torch.float64)
    _check((250, 40001), 0, torch.float64)
    _check((300, 30011), 0, torch.float32)
