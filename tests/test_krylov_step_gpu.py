"""FGMRES where a Gram-Schmidt step on short segments is one launch: segment
lengths below and above each number of entries per thread and the limit
(1,024 threads; 1, 2 or 4 entries each), alone and in a batch of uneven
members, basis sizes below, at and above the groups of eight columns; against
the oracle's FGMRES."""
import numpy as np
import pytest

import oracle
from gpu_common import log, relerr, to_dev, to_host
from stgen.problem import make_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def stv():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    import paper_2107_10561_amd as m
    return m


# segments of 402, 1540, 3012, 3972, 4252 and 7332 (the last two over the limit), and batches of
# three (short) and four (one over the limit, so that all take the separate kernels)
@pytest.mark.parametrize("k,shapes", [(0, [(8, 4)]), (1, [(8, 8)]), (1, [(16, 8)]), (1, [(28, 6)]),
                                      (1, [(30, 6)]), (1, [(20, 16)]),
                                      (1, [(16, 8), (8, 8), (4, 2)]),
                                      (1, [(16, 8), (8, 8), (4, 2), (20, 16)])])
def test_short_segments(stv, k, shapes):
    prob = [make_problem(2, n, 2, k, 0.01, 1e-3, 19 + i) for i, n in enumerate(shapes)]
    s = stv.Solver(0)
    if len(prob) > 1:
        s.set_batch([p.levels for p in prob], 2, k)
    else:
        s.set_hierarchy(prob[0].levels, 2, k)
    s.build_cell_inverses()
    rhs = to_dev(np.concatenate([p.rhs for p in prob]))
    got = {}
    for n in (1, 8, 9, 18):
        x = to_dev(np.zeros(rhs.numel()))
        s.gmres_solve(rhs, x, restart=30, fixed_iters=n, nu1=1, nu2=0)
        got[n] = to_host(x)
    at = 0
    for p in prob:
        ol = oracle.build_inverses(oracle.prepare_levels(p.levels, p.b))
        cinv = oracle.coarse_inverse(ol[0])
        sl = slice(at, at + p.rhs.size)
        at += p.rhs.size
        for n in got:
            ref, _ = oracle.fgmres(lambda v: ol[-1].J @ v, p.rhs,
                                   lambda v: oracle.vcycle(ol, v, 1, 0, 0.7, coarse_inv=cinv),
                                   restart=30, fixed_iters=n)
            e = relerr(got[n][sl], ref)
            log(f"[krylov] segment {p.rhs.size} k={k} steps {n} rel err {e:.2e}")
            assert e <= 1e-10
    s.close()
