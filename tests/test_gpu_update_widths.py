"""The windowed update at every block width up to 16 against the oracle's Algorithm 1.

Iterates after k block iterations at widths of each kernel form (vector below 8,
matrix cores with the width known at run time for 9 .. 15) on row counts that leave
the last tile or wave ragged, with windows open, just closed and spanning two chunks of
iterations; and full solves in FP64 and mixed precision, where shifts freeze at
different iterations. The small lattices deal the shifts to several groups of
work-groups; an odd check interval switches the windows (and the groups) off.

Tolerances as in test_gpu_mfma.py: iterates 1e-11 against the oracle, and the solver's own
bar, the true residual with the oracle operator, at tol.
"""
import numpy as np
import pytest

from gpu_common import to_dev, to_np, torch_gpu
from oracle import oracle as O
from paper_1808_01829_amd.inputs import configs, gaussian_block, random_gauge

pytestmark = pytest.mark.gpu
BC = (1, 1, 1, -1)
MASS = 0.05


def _problem(torch, dims, n, seed):
    from paper_1808_01829_amd import bms
    U, B = random_gauge(dims, 0.5, seed), gaussian_block(dims, n, seed + 1)
    ctx = bms.Context(dims, BC)
    ctx.set_gauge(to_dev(torch, U))
    return bms, ctx, U, B


@pytest.mark.parametrize("interval", [8, 3])
@pytest.mark.parametrize("dims,n,k", [((2, 2, 2, 6), 1, 6), ((4, 4, 4, 4), 1, 9),
                                      ((2, 2, 2, 6), 2, 7), ((4, 4, 2, 6), 3, 10),
                                      ((4, 4, 4, 6), 4, 11), ((2, 2, 4, 6), 5, 4),
                                      ((4, 2, 4, 6), 6, 8), ((4, 4, 4, 6), 7, 5),
                                      ((2, 4, 4, 6), 9, 6), ((4, 4, 4, 4), 11, 9),
                                      ((2, 2, 6, 6), 12, 4), ((4, 4, 2, 6), 13, 7),
                                      ((4, 4, 4, 6), 15, 9)])
def test_update_matches_oracle_iterates(dims, n, k, interval):
    torch = torch_gpu()
    bms, ctx, U, B = _problem(torch, dims, n, 300 + n)
    r = configs.workload_coefficients("c2")
    oo = O.sbcgrq_lattice(dims, BC, U, MASS, r.beta, B, 1e-30, maxiter=k)
    assert oo["iters"] == k
    X, st = ctx.solve(MASS, r.beta, to_dev(torch, B), tol=1e-15, max_iter=k, max_refine=0,
                      check_interval=interval, raise_on_error=False)
    X = to_np(X)
    assert st["iterations"] == k
    for s in range(len(r.beta)):
        err = np.linalg.norm(X[s] - oo["X"][s]) / np.linalg.norm(oo["X"][s])
        assert err <= 1e-11, (s, err)


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("n", [1, 2, 3, 5, 7, 10, 14])
def test_update_widths_solve(n, mixed):
    torch = torch_gpu()
    dims = (4, 6, 4, 6)
    bms, ctx, U, B = _problem(torch, dims, n, 500 + n)
    r = configs.workload_coefficients("c2")
    X, st = ctx.solve(MASS, r.beta, to_dev(torch, B), tol=1e-10,
                      precision=bms.BMS_PREC_MIXED if mixed else bms.BMS_PREC_F64)
    assert O.true_residuals(dims, BC, U, MASS, r.beta, B, to_np(X)).max() <= 1e-10


CLOSE_DIMS = (6, 14, 14, 10)  # 17640 rows: 1102.5 tiles of 16


@pytest.mark.parametrize("n,k", [(8, 4), (8, 7), (12, 4), (12, 11), (16, 2), (16, 9),
                                 (16, 11)])
def test_closed_windows_match_oracle_iterates(n, k):
    torch = torch_gpu()
    bms, ctx, U, B = _problem(torch, CLOSE_DIMS, n, 700 + n)
    r = configs.workload_coefficients("c2")
    oo = O.sbcgrq_lattice(CLOSE_DIMS, BC, U, MASS, r.beta, B, 1e-30, maxiter=k)
    X, st = ctx.solve(MASS, r.beta, to_dev(torch, B), tol=1e-15, max_iter=k, max_refine=0,
                      check_interval=8, raise_on_error=False)
    X = to_np(X)
    assert st["iterations"] == k
    for s in range(len(r.beta)):
        err = np.linalg.norm(X[s] - oo["X"][s]) / np.linalg.norm(oo["X"][s])
        assert err <= 1e-11, (s, err)


@pytest.mark.parametrize("n", [8, 12, 16])
def test_closed_windows_mixed_solve(n):
    torch = torch_gpu()
    bms, ctx, U, B = _problem(torch, CLOSE_DIMS, n, 800 + n)
    r = configs.workload_coefficients("c2")
    X, st = ctx.solve(0.2, r.beta, to_dev(torch, B), tol=1e-10,
                      precision=bms.BMS_PREC_MIXED)
    assert O.true_residuals(CLOSE_DIMS, BC, U, 0.2, r.beta, B, to_np(X)).max() <= 1e-10


@pytest.mark.parametrize("interval", [8, 6, 3])
@pytest.mark.parametrize("dims,n,k", [((4, 4, 4, 6), 17, 6), ((4, 4, 4, 6), 20, 4),
                                      ((4, 4, 6, 6), 24, 9), ((4, 6, 4, 6), 25, 7),
                                      ((4, 6, 4, 6), 31, 5), ((6, 6, 4, 6), 32, 9)])
def test_wide_update_matches_oracle_iterates(dims, n, k, interval):
    test_update_matches_oracle_iterates(dims, n, k, interval)


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("dims,n", [((4, 6, 4, 6), 18), ((4, 6, 6, 6), 24), ((6, 6, 6, 6), 29),
                                    ((8, 8, 8, 8), 32)])
def test_wide_update_solve(dims, n, mixed):
    torch = torch_gpu()
    bms, ctx, U, B = _problem(torch, dims, n, 600 + n)
    r = configs.workload_coefficients("c2")
    X, st = ctx.solve(0.2, r.beta, to_dev(torch, B), tol=1e-10,
                      precision=bms.BMS_PREC_MIXED if mixed else bms.BMS_PREC_F64)
    assert O.true_residuals(dims, BC, U, 0.2, r.beta, B, to_np(X)).max() <= 1e-10
