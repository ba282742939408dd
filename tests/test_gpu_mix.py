"""GPU: the points of a request give the same bits alone and among many others in a launch.

The sizes stand on both sides of what a launch of more matrices may change: workgroups per solve, waves per
residual, tiles of a product, split operands of wide solves.  Oracle: the call alone.
"""
import numpy as np
import pytest
import torch

import workloads as W
from paper_1605_07951_amd import rsrr as R

pytestmark = pytest.mark.gpu


def _nep(n, seed):
    rng = np.random.default_rng(seed)
    A = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)) + 2.0 * np.sqrt(n) * np.eye(n)
    return R.DeviceNEP(W.SeparableNEP(name="mix", A=[A], terms=[W.term(1.0, 1)]))


def _same_alone(n, L, count, prec, N=24):
    ctx = R.rsrr_create(0)
    rng = np.random.default_rng(n + L)
    z = np.exp(2j * np.pi * (np.arange(N) + 0.5) / N)
    first, other = _nep(n, 1), _nep(n, 2)
    items = [R.BatchItem(first if q == 0 else other, z * (1.0 + 0.01 * q),
                         rng.standard_normal((n, L)) + 1j * rng.standard_normal((n, L))) for q in range(count)]
    mixed_info, _ = R.rsrr_sample_batched(ctx, items, prec=prec)
    torch.cuda.synchronize()
    mixed = items[0].S.clone()
    items[0].S.zero_()
    alone_info, _ = R.rsrr_sample_batched(ctx, items[:1], prec=prec)
    torch.cuda.synchronize()
    ctx.close()
    assert mixed_info[0] == alone_info[0]
    assert torch.equal(items[0].S, mixed)


# more than 512 workgroups of 16 right-hand sides in the mix, fewer alone
@pytest.mark.parametrize("n,L,count", [(60, 17, 22), (60, 32, 22), (130, 32, 12), (130, 64, 6), (60, 64, 8)])
def test_solve_kernel(n, L, count):
    _same_alone(n, L, count, R.RSRR_PREC_C64_IR)


def test_wide_solve():
    """256 right-hand sides at a size whose trailing updates are split (2048 over all matrices in the mix)."""
    _same_alone(330, 256, 4, R.RSRR_PREC_C64_IR, N=4)


@pytest.mark.parametrize("n,L,count,prec", [(250, 40, 12, R.RSRR_PREC_C64_IR), (250, 40, 12, R.RSRR_PREC_C128)])
def test_fp64_product_tiles(n, L, count, prec):
    """Enough matrices for 128 x 64 tiles in the mix, 64 x 64 alone."""
    _same_alone(n, L, count, prec)


# 512 blocks of 64 rows and more in the mix, fewer alone
@pytest.mark.parametrize("n,L,count", [(60, 2, 22), (60, 8, 22), (300, 1, 5), (300, 3, 5), (300, 5, 5), (300, 8, 5),
                                       (700, 4, 2), (120, 9, 12), (120, 20, 12)])
@pytest.mark.parametrize("prec", [R.RSRR_PREC_C64_IR, R.RSRR_PREC_C128])
def test_residual(n, L, count, prec):
    _same_alone(n, L, count, prec)
