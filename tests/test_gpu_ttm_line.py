"""FP64 TTM, many output rows of a wide mode: which sizes take the kernel with
the operator in registers, both sides of that line, and the kernel itself at
sizes below it (where its edges are cheap to visit)."""
import ctypes

import pytest
import torch

from paper_1510_06689_amd import tucker

pytestmark = pytest.mark.gpu


class View(ctypes.Structure):
    _fields_ = [("L", ctypes.c_int64), ("B", ctypes.c_int64), ("J", ctypes.c_int)]


def _inputs(l, j, b, k, dtype, transpose):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(3 + j + k)
    y = torch.randn(b, j, l, generator=g, dtype=torch.float64, device="cuda:0").to(dtype)
    m = torch.randn((k, j) if transpose else (j, k), generator=g, dtype=torch.float64, device="cuda:0").t()
    return y, m


def _check(z, y, m, transpose):
    """J products and sums on either side, at most J u |m_r||y_c| each, and one
    rounding to the storage type."""
    op = (m.t() if transpose else m).contiguous()
    j = y.shape[1]
    a = y.double().permute(1, 0, 2).reshape(j, -1)
    ref = op @ a
    got = z.double().permute(1, 0, 2).reshape(op.shape[0], -1)
    bound = 2 * j * 2.0 ** -53 * op.norm(dim=1)[:, None] * a.norm(dim=0)[None, :]
    unit = 2.0 ** -24 if y.dtype == torch.float32 else 2.0 ** -53
    assert bool(((got - ref).abs() <= bound + unit * ref.abs() * (1 + 1e-6)).all())


def _in_registers(y, m, transpose):
    t = "d" if y.dtype == torch.float64 else "f"
    fn = tucker.library()[f"_ZN2tk14launch_ttm_regEPK{t}RKNS_8ModeViewEPKdliiP{t}P12ihipStream_t" if t == "f"
                          else "_ZN2tk14launch_ttm_regEPKdRKNS_8ModeViewES1_liiPdP12ihipStream_t"]
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.c_void_p, ctypes.POINTER(View), ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_int,
                   ctypes.c_void_p, ctypes.c_void_p]
    b, j, l = y.shape
    k = m.shape[1] if transpose else m.shape[0]
    z = torch.full((b, k, l), float("nan"), dtype=y.dtype, device=y.device)
    v = View(l, b, j)
    assert fn(y.data_ptr(), ctypes.byref(v), m.data_ptr(), m.shape[0], k, int(transpose), z.data_ptr(),
              torch.cuda.current_stream().cuda_stream) == 0
    return z


@pytest.mark.parametrize("j", [96, 97, 111, 128, 129, 192, 193, 250, 256])
@pytest.mark.parametrize("k", [33, 64, 65, 100, 129])
def test_operator_in_registers(j, k):
    for l, b, dtype, transpose in [(1, 333, torch.float64, True),     # a partial last tile
                                   (3, 91, torch.float32, True),      # packed, L < 16
                                   (20, 17, torch.float64, False),    # packed, L >= 16, padding columns
                                   (135, 3, torch.float32, False),    # strided
                                   (1, 20003, torch.float32, True)]:  # several tiles per workgroup
        y, m = _inputs(l, j, b, k, dtype, transpose)
        _check(_in_registers(y, m, transpose), y, m, transpose)


@pytest.mark.parametrize("j,k,least", [(96, 40, 8), (111, 200, 8), (112, 64, 3), (192, 33, 3), (193, 64, 6), (193, 65, 3), (256, 129, 3)])
@pytest.mark.parametrize("l", [1, 20, 100])
def test_both_sides_of_the_line(j, k, least, l):
    kt, rows = (64 if j <= 128 else 32), (64 if k <= 64 else 128)
    groups = -(-k // rows)
    per_tile = kt // l if l <= kt else 1            # b-blocks per tile
    tiles_per = 1 if l <= kt else -(-l // kt)       # tiles per b-block
    last_below = least * 256 // groups * per_tile // tiles_per
    for b, inside in ((last_below, False), (last_below + per_tile, True)):
        for dtype in (torch.float64, torch.float32):
            y, m = _inputs(l, j, b, k, dtype, True)
            z = tucker.ttm(y.permute(2, 1, 0), 1, m, True).permute(2, 1, 0)
            _check(z, y, m, True)
            # the two kernels sum in different orders: equal bits tell which one ran
            assert torch.equal(z, _in_registers(y, m, True)) == inside or dtype == torch.float32
