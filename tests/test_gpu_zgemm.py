"""GPU: the complex FP64 GEMM at the edges of its tiles (64 and 128 rows, 64 columns) and stages
(8 inner indices), through the projection Q^H A_j Q (a plain and a Hermitian product).

Oracle: NumPy.  Tolerance: two products of depth n round at most 2 n u relative to the norms.
"""
import ctypes as C

import numpy as np
import pytest
import torch

import workloads as W
from paper_1605_07951_amd import rsrr as R

pytestmark = pytest.mark.gpu

U64 = 2.0**-53


@pytest.fixture(scope="module")
def ctx():
    c = R.rsrr_create(0)
    yield c
    c.close()


def _problem(n, k, J):
    rng = np.random.default_rng(10000 * n + 10 * k + J)
    A = [rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)) for _ in range(J)]
    Q = rng.standard_normal((n, k)) + 1j * rng.standard_normal((n, k))
    return W.SeparableNEP(name="zgemm", A=A, terms=[W.term(1.0, j) for j in range(J)]), Q


def _check(nep, Q, AQ):
    n = Q.shape[0]
    for j, A in enumerate(nep.A):
        ref = Q.conj().T @ A @ Q
        got = AQ[j].cpu().numpy().T
        bound = 2 * max(n, 4) * U64 * np.linalg.norm(A) * np.linalg.norm(Q) ** 2
        assert np.linalg.norm(got - ref) <= bound


@pytest.mark.parametrize("n,k", [(1, 1), (5, 3), (8, 8), (63, 64), (64, 63), (65, 66), (129, 7), (200, 130), (331, 65)])
def test_small_tiles(ctx, n, k):
    nep, Q = _problem(n, min(n, k), 2)
    AQ, _ = R.rsrr_project(ctx, R.DeviceNEP(nep), R.colmajor(Q)[0], Q.shape[1], 0j, 1.0)
    _check(nep, Q, AQ)


@pytest.mark.parametrize("n,k", [(257, 65), (300, 130)])
def test_large_tiles(ctx, n, k):
    """Enough matrices for 128 x 64 tiles."""
    nep, Q = _problem(n, k, 64)
    AQ, _ = R.rsrr_project(ctx, R.DeviceNEP(nep), R.colmajor(Q)[0], k, 0j, 1.0)
    _check(nep, Q, AQ)


def test_operand_aligned_to_8_bytes(ctx):
    """A caller's matrix may start at any double."""
    n, k = 70, 33
    nep, Q = _problem(n, k, 2)
    d = R.DeviceNEP(nep)
    buf = torch.zeros(2 * n * k + 1, dtype=torch.float64, device="cuda")
    buf[1:] = torch.from_numpy(np.ascontiguousarray(Q.T).view(np.float64).ravel())
    AQ = torch.zeros((2, k, k), dtype=torch.complex128, device="cuda")
    J, terms = C.c_int(0), (R.RsrrTerm * 2)()
    g = (C.c_double * 2)(0.0, 0.0)
    torch.cuda.synchronize()
    code = R.lib().rsrr_project(ctx.h, C.byref(d.desc), buf.data_ptr() + 8, n, k, g, 1.0, AQ.data_ptr(), 2,
                                C.byref(J), terms)
    assert code == R.RSRR_OK
    _check(nep, Q, AQ)


@pytest.mark.parametrize("n,k", [(383, 383), (384, 384), (384, 377), (383, 321)])
def test_tiles_of_128_rows(ctx, n, k):
    """Both products on 128 x 64 tiles: at least 512 of them over the matrices, and no more rows padded than
    with 64 x 64 (plain product n x k, Hermitian product k x k)."""
    J = 32
    for rows in (n, k):
        t128, t64 = -(-rows // 128), -(-rows // 64)
        assert t128 * -(-k // 64) * J >= 512 and 2 * t128 * 20 <= t64 * 21
    nep, Q = _problem(n, k, J)
    AQ, _ = R.rsrr_project(ctx, R.DeviceNEP(nep), R.colmajor(Q)[0], k, 0j, 1.0)
    _check(nep, Q, AQ)
