"""GPU: the inverted diagonal blocks of the LU at the edges of their 16-row blocks, in the three element types.

A last panel of jb rows (n = panel width + jb, or jb alone) meets a T whose LU has large
off-diagonal entries in the diagonal blocks; the FP64 result is compared with the host's solution,
the refined ones by their residual and their number of corrections.
"""
import numpy as np
import pytest

import workloads as W
from paper_1605_07951_amd import rsrr as R

pytestmark = pytest.mark.gpu

U64 = 2.0**-53


def _matrix(n, real):
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n)) + (0 if real else 1j) * rng.standard_normal((n, n))
    return A / np.sqrt(n) + 2.5 * np.eye(n)[rng.permutation(n)]


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 33, 48, 63, 65, 80, 81, 127, 128, 129, 143, 145, 161, 191])
@pytest.mark.parametrize("mode", ["c128", "c64", "real"])
def test_diagonal_blocks(n, mode):
    ctx = R.rsrr_create(0)
    A = _matrix(n, mode == "real")
    nep = W.SeparableNEP(name="triinv", A=[A.astype(complex), np.eye(n, dtype=complex)],
                         terms=[W.term(), W.term(1.0, 1)])
    rng = np.random.default_rng(n + 1)
    U = (rng.standard_normal((n, 3)) + (0 if mode == "real" else 1j) * rng.standard_normal((n, 3))).astype(complex)
    z = np.array([0.0, 0.1])
    prec = {"c128": R.RSRR_PREC_C128, "c64": R.RSRR_PREC_C64_IR, "real": R.RSRR_PREC_R32_IR}[mode]
    S, info, status = R.rsrr_sample(ctx, R.DeviceNEP(nep), z, U, prec=prec)
    assert status == R.RSRR_OK
    X = R.from_colmajor(S, n)
    for k in range(2):
        T = A + z[k] * np.eye(n)
        x = X[:, 3 * k:3 * k + 3]
        r = np.linalg.norm(U - T @ x, axis=0)
        den = np.linalg.norm(T) * np.linalg.norm(x, axis=0) + np.linalg.norm(U, axis=0)
        # a backward stable solve: n u with a growth of at most 8
        assert (r / den).max() <= 8 * max(n, 4) * U64
        if mode != "c128":
            # kappa(T) below 50, so a correction gains 2^24 / (8 n 50) > 200: 14 digits take at most 6
            assert info[k]["ir_iters"] <= 6 and not info[k]["fallback"]
    ctx.close()
