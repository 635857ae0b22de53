"""Every column of the half hop with four threads per site, at the widths that take it from 1.5
waves per SIMD on: 3, 5, 6 and 8 columns a thread, single precision in pairs with an odd tail.

The lattices that reach that form are too large to have the oracle on every column, so all columns
are compared with the per-group kernel (variant 0; one, two or four columns a thread, which the
small lattices' tests compare with the oracle in full) and a middle one with the oracle.
Tolerances: a sum of 24 (48) products for each, twice that between them.
"""
import numpy as np
import pytest

from gpu_common import rel, to_dev, to_np, torch_gpu
from oracle import oracle as O
from paper_1808_01829_amd.inputs import gaussian_block, random_gauge

pytestmark = pytest.mark.gpu
BC = (1, -1, 1, -1)


@pytest.mark.parametrize("links", ["two rows", "nine entries", "three-hop"])
@pytest.mark.parametrize("dims", [(12, 16, 16, 16), (14, 16, 16, 14)])
def test_every_column(dims, links):
    torch = torch_gpu()
    from paper_1808_01829_amd import bms
    U = random_gauge(dims, 0.6, 61)
    W = 0.1 * random_gauge(dims, 0.6, 62) if links == "three-hop" else None
    c = bms.Context(dims, BC)
    if W is not None:
        c.set_gauge_improved(to_dev(torch, U), to_dev(torch, W))
    else:
        c.set_link_rows(2 if links == "two rows" else 3)
        c.set_gauge(to_dev(torch, U))
    for n in (12, 20, 24, 32):
        v = gaussian_block(dims, n, 63 + n)
        vd = to_dev(torch, v)
        ref = O.mdagm(dims, BC, U, 0.1, 0.2, np.ascontiguousarray(v[..., n // 2]), W)
        for prec, x, bar in ((bms.BMS_PREC_F64, vd, 1e-13),
                             (bms.BMS_PREC_F32, vd.to(torch.complex64), 2e-6)):
            out = {}
            for variant in (-1, 1, 0):
                c.set_variant(bms.BMS_KERNEL_HOP, variant)
                out[variant] = to_np(c.apply_mdagm(0.1, 0.2, x, prec))
            assert rel(out[-1][..., n // 2], ref) < bar, n
            for j in range(n):
                for variant in (-1, 1):
                    assert rel(out[variant][..., j], out[0][..., j]) < 2 * bar, (n, prec, j)
