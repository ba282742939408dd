"""GPU: the FP64 residual of at most 32 columns at the edges of its row blocks, column
counts and point counts (few points: the columns of T split over more waves).

The refinement only converges on a right residual, and the residual it reports is
compared with the one recomputed on the host.
"""
import numpy as np
import pytest

import workloads as W
from paper_1605_07951_amd import rsrr as R

pytestmark = pytest.mark.gpu

U64 = 2.0**-53


@pytest.fixture(scope="module")
def ctx():
    c = R.rsrr_create(0)
    yield c
    c.close()


def _run(ctx, n, N, L, ldu=0):
    rng = np.random.default_rng(1000 * n + 16 * N + L)
    A = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)) + 3.0 * np.sqrt(n) * np.eye(n)
    nep = W.SeparableNEP(name="resid", A=[A, np.eye(n, dtype=np.complex128)], terms=[W.term(), W.term(1.0, 1)])
    U = rng.standard_normal((n, L)) + 1j * rng.standard_normal((n, L))
    z = 0.1 * np.exp(2j * np.pi * np.arange(N) / N)
    S, info, status = R.rsrr_sample(ctx, R.DeviceNEP(nep), z, U)
    assert status == R.RSRR_OK
    X = R.from_colmajor(S, n)
    for k in sorted({0, 1, N // 2, N - 1} & set(range(N))):
        T = A + z[k] * np.eye(n)
        x = X[:, k * L:(k + 1) * L]
        r = np.linalg.norm(U - T @ x, axis=0)
        den = np.linalg.norm(T) * np.linalg.norm(x, axis=0) + np.linalg.norm(U, axis=0)
        assert (r / den).max() <= 8 * max(n, 4) * U64
        # reported against recomputed: both carry their own rounding, at most n u of the same scale
        rel = (r / np.linalg.norm(U, axis=0)).max()
        assert abs(info[k]["resid"] - rel) <= 8 * max(n, 4) * U64 * (den / np.linalg.norm(U, axis=0)).max()


@pytest.mark.parametrize("L", [1, 2, 3, 4, 5, 8, 9, 15, 16, 17, 31, 32, 33])
@pytest.mark.parametrize("n", [1, 3, 31, 63, 65, 129, 515])
def test_residual_edges(ctx, n, L):
    _run(ctx, n, 3, L)


@pytest.mark.parametrize("L", [1, 3, 7, 16])
def test_residual_many_points(ctx, L):
    """Enough row blocks that four waves share one."""
    _run(ctx, 66, 300, L)
