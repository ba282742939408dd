"""GPU: what a point redone in FP64 costs a ragged batch.

The redo is a call of one point.  It may cost what that call costs alone, not the creation and release of
streams around it (5 ms a batch).
"""
import time

import numpy as np
import pytest
import torch

import workloads as W
from paper_1605_07951_amd import rsrr as R

pytestmark = pytest.mark.gpu


def _matrix(n, seed, graded):
    rng = np.random.default_rng(seed)
    A = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    if not graded:
        return A + 2.0 * np.sqrt(n) * np.eye(n)
    q, _ = np.linalg.qr(A)
    return (q * np.logspace(0, -13, n)[None, :]) @ q.conj().T   # FP32 factors do not refine


def test_cost_of_a_redone_point():
    n, N, L = 200, 8, 4
    ctx = R.rsrr_create(0)
    rng = np.random.default_rng(5)

    def item(seed, graded):
        nep = R.DeviceNEP(W.SeparableNEP(name="redo", A=[_matrix(n, seed, graded)], terms=[W.term(1.0, 1)]))
        return R.BatchItem(nep, np.exp(1j * np.arange(1 if graded else N)),
                           rng.standard_normal((n, L)) + 1j * rng.standard_normal((n, L)))

    rest = [item(s, False) for s in range(3)]
    plain, redone = rest + [item(3, False)], rest + [item(4, True)]
    one = redone[-1]

    def batch(items):
        return lambda: R.rsrr_sample_batched(ctx, items)

    calls = [batch(plain), batch(redone),
             lambda: R.rsrr_sample(ctx, one.dnep, one.z, one.U, prec=R.RSRR_PREC_C128)]
    assert calls[1]()[1] == R.RSRR_WARN_FALLBACK and calls[0]()[1] == R.RSRR_OK
    best = [np.inf] * 3
    for _ in range(10):
        for i, f in enumerate(calls):
            torch.cuda.synchronize()
            t = time.perf_counter()
            f()
            torch.cuda.synchronize()
            best[i] = min(best[i], 1e3 * (time.perf_counter() - t))
    ctx.close()
    # half of what the streams cost as the margin
    assert best[1] <= best[0] + best[2] + 2.5
