"""Reduction of extents above 192 when its waves don't get to run together: a
wave that finds too much missing gives up, and one workgroup does the columns
instead.  The wait is made to end at once by its limit; the result has to be
the same, bit for bit."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1510_06689_amd import tucker

pytestmark = pytest.mark.gpu

KGRIDPOLLS = 1 << 16


def _reduce(s, polls):
    """T with its bounds, the reflectors and what the first area of the scratch holds."""
    lib = tucker.library()
    size = lib["_ZN2tk19eig_scratch_doublesEi"]
    size.restype, size.argtypes = ctypes.c_size_t, [ctypes.c_int]
    reduce = lib["_ZN2tk17launch_eig_reduceEPKdiPdPiiP12ihipStream_t"]
    reduce.restype = ctypes.c_int
    reduce.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    j = s.shape[0]
    scratch = torch.full((size(j),), 7.0, dtype=torch.float64, device="cuda:0")
    flags = torch.zeros(2, dtype=torch.int32, device="cuda:0")
    assert reduce(s.data_ptr(), j, scratch.data_ptr(), flags.data_ptr(), polls, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert flags.tolist() == [0, 0]
    a, h, rest = scratch[: j * j].view(j, j), scratch[j * j: 2 * j * j].view(j, j), scratch[3 * j * j:]
    below = torch.arange(j, device="cuda:0")[:, None] + torch.arange(j, device="cuda:0")[None, :] < j - 1
    below[j - 2:] = False  # reflector k at row k, j - k - 1 entries, k < j - 2
    return torch.where(below, h, 0.0), rest[: 5 * j + 4], a


@pytest.mark.parametrize("j", [193, 200, 255, 256, 257, 301, 321, 400, 512])
def test_one_workgroup_gives_the_same_bits(j):
    x = np.random.default_rng(j).standard_normal((j, j + 3)) * 0.98 ** np.arange(j)[:, None]
    s = torch.from_numpy(x @ x.T).to("cuda:0")
    h0, t0, _ = _reduce(s, KGRIDPOLLS)
    h1, t1, a = _reduce(s, 0)
    assert torch.equal(a[0], s[0])  # the one workgroup ran: its copy of S
    assert bool(torch.isfinite(t0).all())
    assert torch.equal(t0, t1) and torch.equal(h0, h1)
    # d, e: the spectrum of S, to 16 J u |S| for either side
    d, e = t1[:j].cpu().numpy(), t1[j: 2 * j - 1].cpu().numpy()
    lam = np.linalg.eigvalsh(s.cpu().numpy())
    got = np.linalg.eigvalsh(np.diag(d) + np.diag(e, 1) + np.diag(e, -1))
    assert np.abs(got - lam).max() <= 16 * j * 2.0 ** -53 * lam[-1]


def test_zero_couplings():
    s = torch.diag(torch.arange(1.0, 261.0, dtype=torch.float64)).to("cuda:0")  # every reflector is the identity
    h0, t0, _ = _reduce(s, KGRIDPOLLS)
    h1, t1, _ = _reduce(s, 0)
    assert torch.equal(t0, t1) and torch.equal(h0, h1)
    assert torch.equal(t1[:260], s.diagonal())
