"""The register-resident n x n step (n <= 16) against the oracle's Algorithm 1.

Iterates after k block iterations as in test_gpu_mfma.py, at the block widths
where the kernel's layout changes: one to four register rows (n up to 4, 8,
12, 16) with full and ragged last rows. A heavy mass makes V = Q - W alpha
small next to Q, which sends every iteration through the explicit Gram.
Duplicate and far-apart shifts take the recurrence to its two limits
(beta = 1 and beta -> 0).

Tolerance: the iterates amplify rounding by at most the condition number of
the n x n Grams (below 1e3 here) per iteration, 10 x 2.2e-16 x 1e3 = 2e-12 and
k <= 6 of them: 1e-11, the bar of the other iterate tests.
"""
import numpy as np
import pytest

from gpu_common import to_dev, to_np, torch_gpu
from oracle import oracle as O
from paper_1808_01829_amd.inputs import gaussian_block, random_gauge

pytestmark = pytest.mark.gpu
BC = (1, 1, 1, -1)
DIMS = (4, 4, 2, 6)  # 288 rows
SHIFTS = [1e-3, 1e-3, 4e-3, 0.3, 7.0, 250.0]


@pytest.mark.parametrize("mass", [0.05, 30.0])
@pytest.mark.parametrize("n,k", [(1, 6), (2, 5), (3, 4), (4, 4), (5, 6), (7, 3), (8, 6), (9, 4),
                                 (12, 5), (13, 3), (15, 4), (16, 6)])
def test_small_step_matches_oracle_iterates(n, k, mass):
    torch = torch_gpu()
    from paper_1808_01829_amd import bms
    U = random_gauge(DIMS, 0.5, 40 + n)
    B = gaussian_block(DIMS, n, 70 + k)
    if mass > 1:
        k = min(k, 3)  # a few iterations reach rounding there
    oo = O.sbcgrq_lattice(DIMS, BC, U, mass, SHIFTS, B, 1e-30, maxiter=k)
    assert oo["iters"] == k
    ctx = bms.Context(DIMS, BC)
    ctx.set_gauge(to_dev(torch, U))
    X, st = ctx.solve(mass, SHIFTS, to_dev(torch, B), tol=1e-15, max_iter=k, max_refine=0,
                      raise_on_error=False)
    X = to_np(X)
    assert st["iterations"] == k
    for s in range(len(SHIFTS)):
        err = np.linalg.norm(X[s] - oo["X"][s]) / np.linalg.norm(oo["X"][s])
        assert err <= 1e-11, (s, err)


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("timing", [False, True])
@pytest.mark.parametrize("n,interval", [(1, 8), (4, 3), (8, 8), (11, 1), (16, 8), (20, 8)])
def test_paused_iteration_goes_on(n, interval, timing, mixed):
    """At mass 8 the residual falls by more than 100 in an iteration, so the first solve's
    iteration pauses for the explicit Gram (n <= 16) and the chunk is finished by the host;
    a second solve on the context starts again without the fallback kernels."""
    torch = torch_gpu()
    from paper_1808_01829_amd import bms
    U, B = random_gauge(DIMS, 0.3, 900 + n), gaussian_block(DIMS, n, 901 + n)
    ctx = bms.Context(DIMS, BC)
    ctx.set_gauge(to_dev(torch, U))
    ctx.timing(timing)
    Bd = to_dev(torch, B)
    for mass in (8.0, 0.3, 8.0):
        X, st = ctx.solve(mass, SHIFTS, Bd, tol=1e-11, check_interval=interval,
                          precision=bms.BMS_PREC_MIXED if mixed else bms.BMS_PREC_F64)
        tr = O.true_residuals(DIMS, BC, U, mass, SHIFTS, B, to_np(X))
        assert tr.max() <= 1e-11
        assert st["iterations"] < 400
