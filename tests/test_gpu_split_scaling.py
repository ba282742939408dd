"""GPU: products with split FP16 operands where the rows or columns of T differ by many decades.

A row scaling T = D B reaches the factors as L_ik ~ d_i / d_k and U_kj ~ d_k: the small entries of a
row of L meet the large ones of a column of U.  An FP32 factorisation does not see D (the pivots aside), so
neither may the split products: as many corrections as for B, and every component of x right.

Bars: B (Gaussian entries and 2 sqrt(n) on the diagonal) has a condition number of about 10, so an FP32 solve
gains rho <= 10 n u32 <= 7e-4 a correction in every component, and two corrections reach rho^3 <= 4e-10; one
more may confirm the stop.  GMRES with the inverse of T itself as the preconditioner gains as much an iteration:
four reach 1e-10, two more are allowed.
"""
import numpy as np
import pytest

import workloads as W
from paper_1605_07951_amd import rsrr as R

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = R.rsrr_create(0)
    yield c
    c.close()


def _b(n, real=False):
    rng = np.random.default_rng(n)
    G = rng.standard_normal((n, n)) + (0 if real else 1j * rng.standard_normal((n, n)))
    return (G + 2.0 * np.sqrt(n) * np.eye(n)).astype(complex), rng


def _rows(rng, n, kind, d):
    """Sizes of the rows: one half 10^d times the other, or spread over 2 d decades."""
    if kind == "half":
        return np.where(rng.permutation(n) < n // 2, 10.0**d, 1.0)
    return 10.0 ** rng.uniform(-d, d, n)


def _known(A, L, rng, real=False):
    """x with entries of one size and U = A x, formed in extended precision."""
    n = A.shape[0]
    X = rng.uniform(1, 2, (n, L)) * (rng.choice([-1, 1], (n, L)) if real else np.exp(2j * np.pi * rng.random((n, L))))
    X = X.astype(complex)
    return X, (A.astype(np.clongdouble) @ X.astype(np.clongdouble)).astype(complex)


@pytest.mark.parametrize("kind,d", [("half", 8), ("half", 10), ("half", 12), ("spread", 12)])
@pytest.mark.parametrize("n", [384, 513, 640, 1100])
@pytest.mark.parametrize("prec", [R.RSRR_PREC_C64_IR, R.RSRR_PREC_R32_IR])
def test_rows_of_different_size(ctx, n, kind, d, prec):
    real = prec == R.RSRR_PREC_R32_IR
    B, rng = _b(n, real)
    A = _rows(rng, n, kind, d)[:, None] * B
    X, U = _known(A, 3, rng, real)
    nep = W.SeparableNEP(name="rows", A=[A], terms=[W.term(1.0, 1)])
    z = np.array([1.0, -0.5])
    S, info, status = R.rsrr_sample(ctx, R.DeviceNEP(nep), z, U, prec=prec)
    assert status == R.RSRR_OK
    x = R.from_colmajor(S, n)
    for k, zk in enumerate(z):
        assert info[k]["ir_iters"] <= 3
        # the stop is on the norm, which the large rows carry: two corrections, or as few as gave the rest
        bar = 4e-10 if info[k]["ir_iters"] >= 2 else 7e-4
        assert (np.abs(zk * x[:, 3 * k:3 * k + 3] - X) / np.abs(X)).max() <= bar


@pytest.mark.parametrize("n,d", [(400, 10), (700, 12)])
def test_wide_solves_rows_of_different_size(ctx, n, d):
    """256 right-hand sides: the solves' products are split as well."""
    B, rng = _b(n)
    A = _rows(rng, n, "half", d)[:, None] * B
    X, U = _known(A, 256, rng)
    nep = W.SeparableNEP(name="wide", A=[A], terms=[W.term(1.0, 1)])
    z = np.exp(1j * np.arange(8))
    S, info, status = R.rsrr_sample(ctx, R.DeviceNEP(nep), z, U)
    assert status == R.RSRR_OK
    x = R.from_colmajor(S, n)
    for k, zk in enumerate(z):
        assert info[k]["ir_iters"] <= 3
        bar = 4e-10 if info[k]["ir_iters"] >= 2 else 7e-4
        assert (np.abs(zk * x[:, 256 * k:256 * (k + 1)] - X) / np.abs(X)).max() <= bar


@pytest.mark.parametrize("scaled", ["rows", "columns", "both"])
@pytest.mark.parametrize("n", [300, 700])
def test_gmres_preconditioner(ctx, n, scaled):
    """The explicit inverse (formed by wide solves from 384 rows on) and its product with the basis vectors."""
    B, rng = _b(n)
    d = _rows(rng, n, "half", 12) if scaled in ("rows", "both") else np.ones(n)
    t = _rows(rng, n, "half", 12) if scaled in ("columns", "both") else np.ones(n)
    nep = W.SeparableNEP(name="pre", A=[d[:, None] * B * t[None, :]], terms=[W.term(1.0, 1)])
    U = d[:, None] * (rng.standard_normal((n, 8)) + 1j * rng.standard_normal((n, 8)))
    z = np.exp(0.3j * np.arange(8))
    _, infos, code = R.rsrr_sample_gmres(ctx, R.DeviceNEP(nep), z, U, [1.0 + 0j])
    assert code == R.RSRR_OK
    assert max(i["iters"] for i in infos) <= 6


@pytest.mark.parametrize("N,L", [(2, 2), (16, 1), (16, 4)])
def test_gmres_references_with_rows_of_their_own(ctx, N, L):
    """Two references whose rows have different sizes, each at half of the points: solves with the factors (two
    points), the inverse in FP32 (8 columns a reference) and in split slabs (32)."""
    n = 640
    B, rng = _b(n)
    big = rng.permutation(n) < n // 2
    d1, d2 = np.where(big, 1e12, 1.0), np.where(big, 1e10, 1.0)
    nep = W.SeparableNEP(name="refs", A=[d1[:, None] * B, d2[:, None] * B[:, ::-1]],
                         terms=[W.term(-1.0, 1, 1.0), W.term(1.0, 1)])
    U = d1[:, None] * (rng.standard_normal((n, L)) + 1j * rng.standard_normal((n, L)))
    z = np.arange(N) % 2 + 0j
    _, infos, code = R.rsrr_sample_gmres(ctx, R.DeviceNEP(nep), z, U, [0j, 1.0 + 0j])
    assert code == R.RSRR_OK
    assert max(i["iters"] for i in infos) <= 6


def test_weakly_coupled_columns(ctx):
    """Rows of different size in a sparse T with columns that hold their diagonal entry alone."""
    n = 640
    rng = np.random.default_rng(7)
    A = (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))) * (rng.random((n, n)) < 0.01)
    A += np.diag(6 * np.exp(2j * np.pi * rng.random(n)))   # about as large as the rest of its row
    alone = rng.permutation(n)[:n // 4]
    A[:, alone] = 0
    A[alone, alone] = 1
    A *= _rows(rng, n, "spread", 5)[:, None]
    X, U = _known(A, 3, rng)
    nep = W.SeparableNEP(name="weak", A=[A], terms=[W.term(1.0, 1)])
    S, info, status = R.rsrr_sample(ctx, R.DeviceNEP(nep), np.array([1.0 + 0j]), U)
    assert status == R.RSRR_OK
    assert info[0]["ir_iters"] <= 3
    assert (np.abs(R.from_colmajor(S, n) - X) / np.abs(X)).max() <= (4e-10 if info[0]["ir_iters"] >= 2 else 7e-4)


@pytest.mark.parametrize("flags", [0, R.RSRR_BATCH_GRAPH])
def test_batch_rows_of_different_size(ctx, flags):
    """The ragged batch refines at most three times; its padding rows are no rows of T."""
    items, known = [], []
    for n, d in ((390, 0), (400, 10), (447, 12)):
        B, rng = _b(n)
        A = _rows(rng, n, "half", d)[:, None] * B * 1e6
        X, U = _known(A, 3, rng)
        known.append(X)
        nep = R.DeviceNEP(W.SeparableNEP(name="batch", A=[A], terms=[W.term(1.0, 1)]))
        items.append(R.BatchItem(nep, np.exp(1j * np.arange(4)), U))
    for _ in range(3 if flags else 1):
        infos, status = R.rsrr_sample_batched(ctx, items, flags=flags)
        assert status == R.RSRR_OK
        for it, X, info in zip(items, known, infos):
            x = R.from_colmajor(it.S, X.shape[0])
            for k, zk in enumerate(it.z):
                bar = 4e-10 if info[k]["ir_iters"] >= 2 else 7e-4
                assert (np.abs(zk * x[:, 3 * k:3 * k + 3] - X) / np.abs(X)).max() <= bar
            it.S.zero_()


def test_reprobe_from_factors_with_scaled_rows():
    """The scales are kept with a request's factors: the reserve columns are solved without a redo."""
    nep, C, U16 = W.cfg_qep(n=400, N=32, L=16)
    D = _rows(np.random.default_rng(3), 400, "half", 10)
    nep.A = [D[:, None] * A for A in nep.A]
    srv = R.Server(max_slots=1, arena_bytes=8 << 30, batch_bytes=4 << 30)
    try:
        res = srv.wait(srv.submit(R.DeviceNEP(nep), R.colmajor(D[:, None] * U16)[0], C.gamma, C.a, C.b, C.N,
                                  max_eigs=128, L_extra=15), 120.0)
    finally:
        srv.close()
    assert res["reprobes"] == 1
    assert res["fallbacks"] == 0
