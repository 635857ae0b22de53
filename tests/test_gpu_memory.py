"""Solves that fit the card's memory only without the ring of residual blocks that the update
windows need (3 blocks more than updating every iteration in FP64): they run all the same, updating
every iteration, and agree with the solve that has the memory.

The workspace of a solve is measured, the context given back and the rest of the memory taken by
a tensor that leaves less than that, by a good part of the ring (blocks of 805 MB: the card gives
about half a GB more than it reports). Iterates after 6 iterations;
tolerance as in the other iterate tests.
"""
import pytest

from gpu_common import torch_gpu

pytestmark = pytest.mark.gpu
L, N = 32, 32
VH = L ** 4 // 2
BLOCK = VH * 3 * N * 16  # bytes
SHIFTS = [0.01, 0.5, 4.0]


def _free(torch):
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _context(bms, U):
    c = bms.Context((L,) * 4, (1, 1, 1, -1))
    c.set_gauge(U)
    return c


@pytest.mark.parametrize("problems,prec", [(1, 0), (1, 2), (2, 0)])
def test_solve_without_room_for_windows(problems, prec):
    torch = torch_gpu()
    from paper_1808_01829_amd import bms
    dev = torch.device("cuda")
    U = torch.eye(3, dtype=torch.complex128, device=dev).expand(4, L ** 4, 3, 3).contiguous()
    g = torch.Generator(device=dev)
    g.manual_seed(3)
    B = torch.view_as_complex(torch.randn(VH, 3, N, 2, dtype=torch.float64, device=dev,
                                          generator=g))
    X = [torch.zeros((len(SHIFTS), VH, 3, N), dtype=torch.complex128, device=dev)
         for _ in range(problems)]
    o = bms.bms_default_opts()
    o.precision, o.max_refine, o.mixed_switch = prec, 0, 0.0

    def solve(ctxs):
        if problems == 1:
            rc, _ = bms.bms_solve(ctxs[0].h, 0.3, N, SHIFTS, 1e-12, 6, o, B, X[0],
                                  raise_on_error=False)
            return [rc]
        return list(bms.bms_solve_batch([c.h for c in ctxs], [0.3] * problems, [N] * problems,
                                        [SHIFTS] * problems, [1e-12] * problems, [6] * problems,
                                        [o] * problems, [B] * problems, X,
                                        raise_on_error=False)[1])

    for _ in range(2):  # what the first solve of the process costs the runtime aside
        ctxs = [_context(bms, U) for _ in range(problems)]
        before = _free(torch)
        assert solve(ctxs) == [bms.BMS_ENOCONV] * problems
        workspace = before - _free(torch)
    assert workspace > 4 * BLOCK * problems
    ref = X[0].clone()
    del ctxs
    ctxs = [_context(bms, U) for _ in range(problems)]
    leave = workspace - int((1.5 if prec == 0 else 1.0) * BLOCK) * problems
    ballast = torch.empty(_free(torch) - leave, dtype=torch.uint8, device=dev)
    try:
        for x in X:
            x.zero_()
        assert solve(ctxs) == [bms.BMS_ENOCONV] * problems
    finally:
        del ballast
        torch.cuda.empty_cache()
    for x in X:
        for s in range(len(SHIFTS)):
            err = ((x[s] - ref[s]).norm() / ref[s].norm()).item()
            assert err < (1e-11 if prec == 0 else 1e-5), (s, err)
    # with the memory back, the next solve has its windows again
    assert solve(ctxs) == [bms.BMS_ENOCONV] * problems
    assert before - _free(torch) > 4 * BLOCK * problems
    assert torch.equal(X[0], ref)
