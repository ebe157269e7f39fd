"""Coarse members cut into parts: regrouping on one solver, parts that cannot
be trusted, batches of members far apart in order."""
import functools

import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as sla

from gpu_common import log, relerr, to_dev, to_host
from stgen import fe as fe_time
from stgen.problem import make_problem, spatial_factors

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def stv():
    import paper_2107_10561_amd as m
    return m


@functools.lru_cache(maxsize=None)
def mesh_problem(dim, n, levels, k):
    return make_problem(dim, n, levels, k, 0.01, 1e-3, 7)


def matrix(L, val, b):
    return sp.bsr_matrix((val, L.col, L.rowptr), shape=(L.n_sdofs * b,) * 2).tocsc()


def check_solve(J, r, d, what):
    """The bounds of every coarse schedule: relative residual, forward error."""
    lu = sla.splu(J)
    cond = sla.onenormest(J) * sla.onenormest(
        sla.LinearOperator(J.shape, matvec=lu.solve, rmatvec=lambda v: lu.solve(v, trans="T")))
    res = np.linalg.norm(r - J @ d) / np.linalg.norm(r)
    fe = relerr(d, lu.solve(r))
    log(f"[coarse] {what} relres {res:.2e} forward {fe:.2e} cond {cond:.1e}")
    assert res <= 1e-11 * max(1.0, 1e-8 * cond)
    assert fe <= 1e-15 * cond * 10


def coarse_solve(s, r):
    dd = to_dev(np.zeros_like(r))
    s.coarse_solve(to_dev(r), dd)
    return to_host(dd)


@pytest.mark.parametrize("then", ["shallow", "prescribed"])
def test_cut_members_and_then_none(stv, then):
    """One solver: a batch whose coarse members are cut on packed levels 0 and
    2, then a hierarchy of two levels whose coarse member is not cut (too small
    without factors), or the same batch with a prescribed schedule."""
    s = stv.Solver(0)
    deep, flat = mesh_problem(2, (64, 16), 3, 1), mesh_problem(2, (16, 4), 1, 1)
    s.set_batch([deep.levels, flat.levels], 2, 1)
    s.build_cell_inverses()
    if then == "shallow":
        p = mesh_problem(2, (8, 2), 2, 1)
        s.set_hierarchy(p.levels, 2, 1)
    else:
        p = deep
        s.set_coarse_algorithm("tournament")
    L = p.levels[0]
    J = matrix(L, L.val, p.b)
    r = np.random.default_rng(3).standard_normal(J.shape[0])
    for _ in range(2):
        s.build_cell_inverses()
        check_solve(J, r, coarse_solve(s, r), then)
    s.close()
