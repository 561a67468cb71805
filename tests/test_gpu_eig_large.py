"""Eigensolver of extents above 128: the reduction over many single-wave
workgroups, its hand-over to the 128 x 128 register reduction and the edges
of its 64-wide row and column slots."""
import numpy as np
import pytest
import torch

from paper_1510_06689_amd import tucker

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def _check(x, r):
    """Spectrum and leading vectors of x x^T (x: J x M) against LAPACK's.

    The computed spectrum is that of a matrix within about J u |S| of S
    (Householder reduction, FP64 Gram); 16 J u covers both sides."""
    j = x.shape[0]
    d = tucker.empty_fortran(x.shape, torch.float64, "cuda:0").copy_(torch.from_numpy(x))
    t = tucker.sthosvd(d, 0.0, ranks=(r, min(x.shape)))
    s = x @ x.T
    lam = np.linalg.eigvalsh(s)[::-1]
    tol = 16 * j * U * lam[0]
    got = t.eigvals[0].cpu().numpy()
    assert np.abs(got - lam).max() <= tol
    u = t.factors[0].cpu().numpy()
    assert np.abs(u.T @ u - np.eye(r)).max() <= 16 * j * U
    assert np.abs(s @ u - u * got[:r]).max() <= 4 * tol


@pytest.mark.parametrize("j", [129, 130, 191, 192, 193, 255, 256, 257, 320, 321, 449, 512])
def test_spectrum_and_vectors(j):
    rng = np.random.default_rng(j)
    q, _ = np.linalg.qr(rng.standard_normal((j, j)))
    x = q * 0.97 ** np.arange(j)          # separated, decaying singular values
    _check(x, 5)


@pytest.mark.parametrize("j", [129, 200, 257])
def test_diagonal_and_rank_deficient(j):
    _check(np.diag(1.0 + np.arange(j, dtype=float)), 3)   # every reflector is the identity
    rng = np.random.default_rng(j)
    q, _ = np.linalg.qr(rng.standard_normal((j, 7)))
    _check(q * np.arange(7, 0, -1), 4)                    # all but seven eigenvalues are zero


def test_nonfinite_input_ends():
    x = np.random.default_rng(0).standard_normal((150, 20))
    x[140, 3] = np.nan
    d = tucker.empty_fortran(x.shape, torch.float64, "cuda:0").copy_(torch.from_numpy(x))
    with pytest.raises(tucker.TuckerError) as err:
        tucker.sthosvd(d, 1e-4)
    assert "NONFINITE" in str(err.value)


@pytest.mark.parametrize("j,r,steps", [
    (64, 43, 1), (64, 64, 1), (97, 29, 1), (128, 22, 1), (128, 128, 1),     # just past one workgroup's batch, and all
    (129, 17, 1), (193, 160, 1), (250, 100, 1), (257, 129, 1), (385, 96, 1),  # registers, their limits and past them
    (150, 40, 5), (300, 33, 11),                                            # clusters with gaps in between
])
def test_many_vectors(j, r, steps):
    """Ranks beyond one workgroup of inverse iteration: Gram-Schmidt inside
    clusters (eigenvalues in groups of `steps`, 1e-4 apart inside one and
    clearly apart from the next; with steps = 1 one slow decay) and the
    back-transformation over several workgroups."""
    rng = np.random.default_rng(1000 * j + r)
    q, _ = np.linalg.qr(rng.standard_normal((j, j)))
    k = np.arange(j)
    lam = 0.995 ** k if steps == 1 else 0.9 ** (k // steps) * (1 + 1e-4 * (steps - k % steps))
    _check(q * np.sqrt(lam), r)
