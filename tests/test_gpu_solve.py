"""GPU: the FP32 solve of at most 64 right-hand sides in one workgroup per 16 and matrix, at the edges of
its panels, row blocks and right-hand-side blocks and on both sides of its size limit.

T = diagonally dominant, so that kappa(T) is below 4 and a right FP32 solve leaves a relative
error of at most about n 2^-24 kappa < 5e-4: the refinement to about 1e-14 then needs at most 4
corrections (5e-4 to the fourth power is 6e-14, to the fifth 3e-17).
"""
import numpy as np
import pytest

import workloads as W
from paper_1605_07951_amd import rsrr as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,L", [(15, 8), (16, 9), (17, 1), (127, 8), (128, 16), (144, 8), (145, 9), (256, 7),
                                 (257, 8), (385, 16), (1024, 16), (1025, 16), (1100, 3), (2048, 8), (2049, 8),
                                 (1, 17), (130, 17), (131, 32), (300, 33), (513, 49), (1024, 64), (1025, 64), (600, 65)])
def test_whole_solve(n, L):
    ctx = R.rsrr_create(0)
    rng = np.random.default_rng(100 * n + L)
    # row interchanges inside and across panels: a permuted dominant matrix
    A = (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))) / (8.0 * np.sqrt(n)) + np.eye(n)
    A = A[rng.permutation(n)]
    nep = W.SeparableNEP(name="solve", A=[A, np.eye(n, dtype=np.complex128)], terms=[W.term(), W.term(1.0, 1)])
    U = rng.standard_normal((n, L)) + 1j * rng.standard_normal((n, L))
    z = np.array([0.0, 0.01, 0.01j])
    S, info, status = R.rsrr_sample(ctx, R.DeviceNEP(nep), z, U)
    assert status == R.RSRR_OK
    X = R.from_colmajor(S, n)
    for k in range(3):
        assert info[k]["ir_iters"] <= 4 and not info[k]["fallback"]
        x = np.linalg.solve(A + z[k] * np.eye(n), U)
        got = X[:, k * L:(k + 1) * L]
        assert np.linalg.norm(got - x) <= 1e-9 * np.linalg.norm(x)
    ctx.close()


@pytest.mark.parametrize("n,L", [(1, 1), (15, 16), (17, 17), (128, 4), (145, 33), (385, 16), (1024, 64), (2048, 16),
                                 (2049, 3), (300, 65)])
def test_whole_solve_real(n, L):
    ctx = R.rsrr_create(0)
    rng = np.random.default_rng(100 * n + L)
    A = rng.standard_normal((n, n)) / (8.0 * np.sqrt(n)) + np.eye(n)
    A = A[rng.permutation(n)]
    nep = W.SeparableNEP(name="solve", A=[A.astype(complex), np.eye(n, dtype=np.complex128)],
                         terms=[W.term(), W.term(1.0, 1)])
    U = rng.standard_normal((n, L)).astype(complex)
    z = np.array([0.0, 0.01, -0.01])
    S, info, status = R.rsrr_sample(ctx, R.DeviceNEP(nep), z, U, prec=R.RSRR_PREC_R32_IR)
    assert status == R.RSRR_OK
    X = R.from_colmajor(S, n)
    for k in range(3):
        assert info[k]["ir_iters"] <= 4 and not info[k]["fallback"]
        x = np.linalg.solve(A + z[k] * np.eye(n), U)
        got = X[:, k * L:(k + 1) * L]
        assert np.linalg.norm(got - x) <= 1e-9 * np.linalg.norm(x)
    ctx.close()
