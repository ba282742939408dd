"""GPU: the panel factorisation at the edges of its row and column ranges.

The base kernel of the LU changes its shape with the rows left (256, 512, 1024,
2048, 4096) and takes 32 columns in groups of 8; the sizes below sit on both
sides of those edges.  Oracle: the FP64 residual on the host.
"""
import numpy as np
import pytest
import torch

import workloads as W
from paper_1605_07951_amd import rsrr as R

pytestmark = pytest.mark.gpu

U64 = 2.0**-53
PRECS = {"c64": R.RSRR_PREC_C64_IR, "c128": R.RSRR_PREC_C128, "r32": R.RSRR_PREC_R32_IR}


@pytest.fixture(scope="module")
def ctx():
    c = R.rsrr_create(0)
    # a point is not handed to the FP64 path for a large ||u - T x|| / ||u||, which an ill-conditioned
    # T gives with any arithmetic: the refined result itself is looked at, by its backward error
    R.rsrr_set_options(c, fallback_resid=0.5)
    yield c
    c.close()


def _nep(A):
    return W.SeparableNEP(name="panel", A=[A, np.eye(A.shape[0], dtype=np.complex128)],
                          terms=[W.term(), W.term(1.0, 1)])


def _check(ctx, A, prec, L=3):
    n = A.shape[0]
    rng = np.random.default_rng(n)
    U = rng.standard_normal((n, L)).astype(np.complex128)
    z = np.array([0.25, -0.5], dtype=np.complex128)
    S, info, status = R.rsrr_sample(ctx, R.DeviceNEP(_nep(A)), z, U, prec=PRECS[prec])
    torch.cuda.synchronize()
    assert status == R.RSRR_OK and all(i["info"] == 0 and i["fallback"] == 0 for i in info)
    X = R.from_colmajor(S, n)
    for k, zk in enumerate(z):
        T = A + zk * np.eye(n)
        x = X[:, k * L:(k + 1) * L]
        r = np.linalg.norm(U - T @ x, axis=0)
        # normwise backward error of a factorisation with partial pivoting (or of its refinement,
        # which stops at 4 u sqrt(n)), with the host residual's own rounding: n u and a constant
        eta = r / (np.linalg.norm(T) * np.linalg.norm(x, axis=0) + np.linalg.norm(U, axis=0))
        assert eta.max() <= 8 * max(n, 4) * U64, (n, prec, eta.max())


@pytest.mark.parametrize("prec", ["c64", "c128", "r32"])
@pytest.mark.parametrize("n", [1, 2, 7, 9, 31, 33, 63, 65, 127, 129, 255, 257, 511, 513, 1023, 1025, 2047, 2049])
def test_panel_edges(ctx, n, prec):
    rng = np.random.default_rng(100 + n)
    A = rng.standard_normal((n, n)).astype(np.complex128)
    if prec != "r32":
        A = A + 1j * rng.standard_normal((n, n))
    _check(ctx, A + 0.1 * np.sqrt(n) * np.eye(n), prec)


@pytest.mark.parametrize("prec", ["c64", "c128", "r32"])
@pytest.mark.parametrize("n", [4097, 4161])
def test_panel_tall(ctx, n, prec):
    """More rows than 4096: the narrowest bases (several per block of 32 columns)."""
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n)).astype(np.complex128)
    _check(ctx, A + 0.1 * np.sqrt(n) * np.eye(n), prec, L=2)


@pytest.mark.parametrize("prec", ["c64", "c128", "r32"])
@pytest.mark.parametrize("n", [40, 200, 300, 700])
def test_panel_ties(ctx, n, prec):
    """Columns with few entries and equal magnitudes: every search has ties, most rows are zero."""
    rng = np.random.default_rng(n)
    A = np.zeros((n, n), dtype=np.complex128)
    A[rng.permutation(n), np.arange(n)] = rng.choice([-4.0, 4.0], n)
    A[rng.permutation(n), np.arange(n)] += rng.choice([-1.0, 1.0], n)
    _check(ctx, A, prec)


@pytest.mark.parametrize("prec", ["c64", "c128"])
@pytest.mark.parametrize("n,col", [(50, 0), (50, 31), (50, 32), (300, 150), (300, 299)])
def test_panel_singular(ctx, n, col, prec):
    """The first exactly zero pivot is reported by its column, as getrf does."""
    rng = np.random.default_rng(col)
    A = rng.standard_normal((n, n)).astype(np.complex128)
    A[:, col] = 0
    nep = W.SeparableNEP(name="singular", A=[A], terms=[W.term()])
    U = np.ones((n, 2), dtype=np.complex128)
    _, info, status = R.rsrr_sample(ctx, R.DeviceNEP(nep), np.array([1.0 + 0j]), U, prec=PRECS[prec],
                                    ok=(R.RSRR_ESINGULAR,))
    assert status == R.RSRR_ESINGULAR and info[0]["info"] == col + 1
