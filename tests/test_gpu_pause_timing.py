"""Per-kernel times of a solve with a paused iteration.

At a heavy mass an iteration of the first pass pauses for the explicit Gram and the host finishes the chunk.
With 64 iterations to a chunk the launches after the pause, which do nothing, take more than
63 x 4 x 1 us before the host sees it, and none of that is time of a kernel: the hops
and Grams (the small step and the update have other work there) take the time they take in
four iterations that do not pause (mass 0.1), half of it and 5 us aside.
"""
import pytest

from gpu_common import to_dev, torch_gpu
from paper_1808_01829_amd.inputs import gaussian_block, random_gauge

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 4, 8, 11, 16])
@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("mass", [8.0, 30.0])
def test_pause_is_no_kernels_time(n, mixed, mass):
    torch = torch_gpu()
    from paper_1808_01829_amd import bms
    dims = (4, 4, 2, 6)
    ctx = bms.Context(dims, (1, 1, 1, -1))
    ctx.set_gauge(to_dev(torch, random_gauge(dims, 0.3, 900 + n)))
    B = to_dev(torch, gaussian_block(dims, n, 901 + n))
    kw = dict(tol=1e-11, check_interval=64, raise_on_error=False,
              precision=bms.BMS_PREC_MIXED if mixed else bms.BMS_PREC_F64)
    shifts = [1e-3, 0.3, 250.0]

    def per_launch(mass, **more):
        ctx.timing(False)
        ctx.solve(mass, shifts, B, **kw, **more)  # allocations and first launches
        best = {}
        for _ in range(5):  # the least of five: a launch that reached an idle GPU late is longer
            ctx.timing(True)
            _, st = ctx.solve(mass, shifts, B, **kw, **more)
            t = ctx.timing_read()
            assert t["hop"][1] == 2 * st["iterations"] and t["gram"][1] == st["iterations"]
            assert t["update"][1] == st["iterations"] and t["cholqr_gram"][1] == st["iterations"]
            for k in ("hop", "gram"):
                best[k] = min(best.get(k, 1e9), t[k][0] / t[k][1])
        return best

    ref = per_launch(0.1, max_iter=4, max_refine=0)
    paused = per_launch(mass)
    for k in ref:
        assert paused[k] < 1.5 * ref[k] + 0.005, (k, paused, ref)
