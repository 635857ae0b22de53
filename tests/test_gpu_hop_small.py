"""The half hop's small-launch forms (a wave per work-group, a batch of hops in flight)
against the oracle, at the widths with 1, 2, 4 and 8 columns a thread, four threads per
site and one per column group, with two-row, nine-entry and three-hop links; on lattices of
less than a wave, with a last wave that is not full, and either side of where the batch
(one wave per SIMD) and the single-wave work-groups end.

Tolerances: a sum of 24 (48 with three-hop links) products, as in test_gpu_operator.py.
"""
import numpy as np
import pytest

from gpu_common import rel, to_dev, to_np, torch_gpu
from oracle import oracle as O
from paper_1808_01829_amd.inputs import gaussian_block, random_gauge

pytestmark = pytest.mark.gpu
BC = (1, -1, 1, -1)


@pytest.mark.parametrize("dims,widths", [((2, 2, 2, 4), (1, 3, 4, 16)), ((4, 6, 4, 6), range(1, 10)),
                                         ((6, 10, 4, 4), (4, 8, 12, 16, 20, 32)),
                                         ((8, 8, 8, 8), (1, 4, 5, 6, 8, 16)),
                                         ((16, 16, 16, 8), (4,)), ((16, 16, 16, 10), (4, 8)),
                                         ((12, 16, 16, 16), (1, 12, 16)),
                                         ((16, 16, 16, 32), (2, 8)), ((16, 16, 16, 34), (4, 8))])
@pytest.mark.parametrize("links", ["two rows", "nine entries", "three-hop"])
def test_small_hop(dims, widths, links):
    torch = torch_gpu()
    from paper_1808_01829_amd import bms
    if links == "three-hop" and min(dims) < 4:
        pytest.skip("three-hop links need extents of 4")
    big = int(np.prod(dims)) > 20000
    U = random_gauge(dims, 0.6, 61)
    W = 0.1 * random_gauge(dims, 0.6, 62) if links == "three-hop" else None
    c = bms.Context(dims, BC)
    if W is not None:
        c.set_gauge_improved(to_dev(torch, U), to_dev(torch, W))
    else:
        c.set_link_rows(2 if links == "two rows" else 3)
        c.set_gauge(to_dev(torch, U))
    for n in widths:
        v = gaussian_block(dims, n, 63 + n)
        cols = range(n) if not big else sorted({0, n - 1})
        ref = np.stack([O.mdagm(dims, BC, U, 0.1, 0.2, np.ascontiguousarray(v[..., j]), W)
                        for j in cols], axis=-1)
        out = to_np(c.apply_mdagm(0.1, 0.2, to_dev(torch, v)))[..., list(cols)]
        assert rel(out, ref) < 1e-13, n
        out = to_np(c.apply_mdagm(0.1, 0.2, to_dev(torch, v.astype(np.complex64)),
                                  bms.BMS_PREC_F32))[..., list(cols)]
        assert rel(out, ref) < 2e-6, n


# 3, 5 and 6 columns a thread: four threads per site from 1.5 waves per SIMD on, the widths'
# other form just below; and eight in single precision (pairs of columns).
@pytest.mark.parametrize("dims", [(12, 16, 16, 16), (14, 16, 16, 14), (12, 16, 16, 14)])
@pytest.mark.parametrize("links", ["two rows", "nine entries", "three-hop"])
def test_four_threads_per_site(dims, links):
    test_small_hop(dims, (12, 20, 24, 32), links)


# One, two and four columns a thread of the per-group form, on either side of the lines
# between them (half a wave per SIMD, a quarter in single precision).
@pytest.mark.parametrize("dims,widths", [((8, 8, 8, 8), (2, 10, 12, 24)),
                                         ((12, 12, 12, 12), (6, 10, 12, 24)),
                                         ((12, 12, 12, 14), (6, 12, 20))])
@pytest.mark.parametrize("links", ["two rows", "nine entries", "three-hop"])
def test_columns_of_a_thread(dims, widths, links):
    test_small_hop(dims, widths, links)
