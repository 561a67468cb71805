"""Sturm counts of the eigensolver: blocks of eight rows read one block ahead
with a remainder of 0 to 7, from LDS (extents below 64) and from the hand-off
of a split solve (64 and up), on spectra that make minors vanish."""
import numpy as np
import pytest
import torch

from paper_1510_06689_amd import tucker

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def _spectrum(x):
    """The computed spectrum is that of a matrix within about J u |S| of S = x x^T;
    16 J u covers both sides."""
    j = x.shape[0]
    d = tucker.empty_fortran(x.shape, torch.float64, "cuda:0").copy_(torch.from_numpy(x))
    got = tucker.sthosvd(d, 0.0, ranks=(1, 1)).eigvals[0].cpu().numpy()
    lam = np.linalg.eigvalsh(x @ x.T)[::-1]
    assert np.abs(got - lam).max() <= 16 * j * U * max(lam[0], 1e-300)


@pytest.mark.parametrize("j", [*range(1, 19), 31, 32, 33, 47, 63, *range(64, 82), 127, 128, 136, 250])
def test_remainders(j):
    rng = np.random.default_rng(j)
    q, _ = np.linalg.qr(rng.standard_normal((j, j)))
    _spectrum(q * 0.9 ** np.arange(j))


@pytest.mark.parametrize("j", [9, 17, 50, 72, 81, 128, 150])
def test_vanishing_couplings(j):
    _spectrum(np.diag(2.0 ** -np.arange(j, dtype=float)))       # every off-diagonal is zero
    _spectrum(np.eye(j))                                        # one eigenvalue J times
    rng = np.random.default_rng(j)
    _spectrum(np.outer(rng.standard_normal(j), rng.standard_normal(j)))  # all but one are zero
    _spectrum(rng.standard_normal((j, j)) * 10.0 ** -rng.integers(0, 12, (j, 1)))  # graded rows


@pytest.mark.parametrize("j,r", [(144, 9), (145, 7), (159, 4), (161, 5), (176, 6), (177, 8), (208, 3), (15, 15), (16, 5), (17, 17), (33, 20), (48, 11), (95, 9), (96, 30), (97, 3), (113, 40), (128, 12)])
def test_reduction_blocks(j, r):
    """Two rows per thread (above 128 rows three), columns in blocks of 16: vectors at the
    blocks' edges, with rows of zeros among them.  |S u - u lambda| is bounded by
    the backward error of the solve, 16 J u |S| on either side as above."""
    rng = np.random.default_rng(7 * j + r)
    q, _ = np.linalg.qr(rng.standard_normal((j, j)))
    x = q * 0.9 ** np.arange(j)
    x[:, : j // 3] *= np.arange(j)[:, None] % 3 != 1
    s = x @ x.T
    d = tucker.empty_fortran(x.shape, torch.float64, "cuda:0").copy_(torch.from_numpy(x))
    t = tucker.sthosvd(d, 0.0, ranks=(r, j))
    got, u = t.eigvals[0].cpu().numpy(), t.factors[0].cpu().numpy()
    lam = np.linalg.eigvalsh(s)[::-1]
    tol = 16 * j * U * lam[0]
    assert np.abs(got - lam).max() <= tol
    assert np.abs(u.T @ u - np.eye(r)).max() <= 16 * j * U
    assert np.abs(s @ u - u * got[:r]).max() <= 4 * tol


@pytest.mark.parametrize("j", [1, 2, 3, 4, 5, 7, 8, 9, 16, 17, 40, 63, 64, 65, 90, 127, 128, 129, 170])
@pytest.mark.parametrize("kind", ["decay", "middle", "twice"])
def test_vectors_from_two_ends(j, kind):
    """Inverse iteration eliminates from both ends and meets in the middle: every
    parity and padding of a half; an entry alone in the middle; the same block on
    either side of it, so that every eigenvalue comes twice.  Residual and
    orthogonality bounds as above."""
    rng = np.random.default_rng(31 * j + len(kind))
    if kind == "twice" and j >= 4:
        m = j // 2
        q, _ = np.linalg.qr(rng.standard_normal((m, m)))
        b = q * 0.8 ** np.arange(m)
        x = np.zeros((j, j))
        x[:m, :m] = b
        x[j - m:, j - m:] = b
    else:
        q, _ = np.linalg.qr(rng.standard_normal((j, j)))
        x = q * 0.9 ** np.arange(j)
        if kind == "middle":
            x[j // 2] = 0.0
            x[j // 2, j // 2] = 1.5
    r = min(j, 14)
    s = x @ x.T
    d = tucker.empty_fortran(x.shape, torch.float64, "cuda:0").copy_(torch.from_numpy(x))
    t = tucker.sthosvd(d, 0.0, ranks=(r, j))
    got, u = t.eigvals[0].cpu().numpy(), t.factors[0].cpu().numpy()
    lam = np.linalg.eigvalsh(s)[::-1]
    tol = 16 * j * U * lam[0]
    assert np.abs(got - lam).max() <= tol
    assert np.abs(u.T @ u - np.eye(r)).max() <= 16 * j * U
    assert np.abs(s @ u - u * got[:r]).max() <= 4 * tol
