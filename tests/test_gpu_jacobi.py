"""GPU: the Jacobi SVD behind rsrr_basis at the edges of its column blocks (16) and row slices.

NL >= 2 rank takes the rotations of R^H without accumulating them, NL < 2 rank the
accumulated form; a truncation below the rotations' zero threshold falls back to the
accumulated form.  Oracle: NumPy's SVD of the normalised matrix.
"""
import numpy as np
import pytest

from paper_1605_07951_amd import rsrr as R

pytestmark = pytest.mark.gpu

EPS = 2.220446049250313e-16


@pytest.fixture(scope="module")
def ctx():
    c = R.rsrr_create(0)
    yield c
    c.close()


def _gauss(rng, shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


def _matrix(n, NL, r, low):
    rng = np.random.default_rng(1000 * n + NL + r)
    X, _ = np.linalg.qr(_gauss(rng, (n, r)))
    Y, _ = np.linalg.qr(_gauss(rng, (NL, r)))
    return (X * np.logspace(0, low, r)[None, :]) @ Y.conj().T


def _check(ctx, S, delta, rank=None):
    n, NL = S.shape
    Q, k, sigma = R.rsrr_basis(ctx, R.colmajor(S)[0], n, delta)
    Sn = S / np.linalg.norm(S, axis=0)
    W, so, _ = np.linalg.svd(Sn, full_matrices=False)
    assert np.abs(sigma - so[:sigma.size]).max() <= 1e-13 * so[0]
    if rank is not None:
        assert k == rank
    Qh = R.from_colmajor(Q, n)[:, :k]
    # pairs of columns are orthogonal to 4 sqrt(NL) eps (the sweeps' stop), their products with the
    # basis of the range round at most with its dimension
    tol = 8 * np.sqrt(NL) * EPS + 4 * min(n, NL) * EPS
    assert np.abs(Qh.conj().T @ Qh - np.eye(k)).max() <= tol
    left = Sn - Qh @ (Qh.conj().T @ Sn)
    assert np.linalg.norm(left, 2) <= max(delta * 1.01, 1e-13) * so[0]


@pytest.mark.parametrize("r", [1, 2, 15, 16, 17, 31, 32, 33, 48, 63, 65, 100])
def test_basis_direct(ctx, r):
    _check(ctx, _matrix(150, 2 * r + 40, r, -5), 1e-9, rank=r)


@pytest.mark.parametrize("n,NL", [(16, 17), (33, 40), (64, 64), (65, 80), (130, 97)])
def test_basis_accumulated(ctx, n, NL):
    """Full rank: NL < 2 r."""
    _check(ctx, _matrix(n, NL, min(n, NL), -3), 1e-8, rank=min(n, NL))


@pytest.mark.parametrize("delta", [1e-14, 1e-16])
def test_basis_truncation_at_rounding(ctx, delta):
    """Singular values down to 1e-16: the smallest kept ones lie at or below the rotations' zero
    threshold, the basis is orthonormal all the same."""
    _check(ctx, _matrix(200, 400, 120, -16), delta)
