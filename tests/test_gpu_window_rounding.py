"""Rounding of the windowed update: a shift far above sigma_0 is nearly solved by the first
iteration, so the sum of its window is one large term, P Cx, and small ones. Added
to last, the large term costs the rounding of one product of n columns; added to first,
every later term of the window is rounded at its size too (eight iterations in FP32 blocks:
up to 2.7 times the error).

FP32 blocks from the start (mixed_switch 0), k iterations, X against the FP64 oracle's
iterate k. Tolerance, for a sum of 2 n products per real part with rms unit rounding
u = 2^-24 / sqrt(3): the coefficients and Q are rounded once each (sqrt 2 u), and the partial
sums, growing like a random walk, add u sqrt(2 n / 2).
"""
import numpy as np
import pytest

from gpu_common import to_dev, to_np, torch_gpu
from oracle import oracle as O
from paper_1808_01829_amd.inputs import gaussian_block, random_gauge

pytestmark = pytest.mark.gpu
BC = (1, 1, 1, -1)
DIMS = (4, 6, 4, 6)
SHIFTS = [1e-3, 0.1, 10.0]


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 9, 10, 12, 13, 15, 17, 20, 24, 25, 31, 32])
def test_large_shift_in_fp32_windows(n):
    torch = torch_gpu()
    from paper_1808_01829_amd import bms
    k = 16 if n < 17 else 12  # whole windows
    U, B = random_gauge(DIMS, 0.5, 7), gaussian_block(DIMS, n, 100 * n)
    oo = O.sbcgrq_lattice(DIMS, BC, U, 0.1, SHIFTS, B, 1e-30, maxiter=k)
    ctx = bms.Context(DIMS, BC)
    ctx.set_gauge(to_dev(torch, U))
    X, st = ctx.solve(0.1, SHIFTS, to_dev(torch, B), tol=1e-15, max_iter=k, max_refine=0,
                      raise_on_error=False, precision=bms.BMS_PREC_MIXED, mixed_switch=0.0)
    assert st["iterations"] == k
    err = np.linalg.norm(to_np(X)[2] - oo["X"][2]) / np.linalg.norm(oo["X"][2])
    assert err <= 2.0 ** -24 / 3 ** 0.5 * (2 ** 0.5 + n ** 0.5), err
