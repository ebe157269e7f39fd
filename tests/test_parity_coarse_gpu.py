"""Dense coarse-level inversion (the direct solve of Algorithm 4.1) through the
C ABI, every elimination schedule, at orders that cover every panel
configuration of the library (up to 8934 unknowns) and ragged padding.
The tournament schedule may take other pivots than partial pivoting: it is
held to the same residual and forward-error bounds.

Expected values: SuperLU applied to the oracle's coarse matrix (a library
routine on the same matrix), and the residual r - J d computed on the CPU."""
import functools

import numpy as np
import pytest
import scipy.sparse.linalg as sla

import oracle
from gpu_common import log, relerr, to_dev, to_host
from stgen import fe as fe_time
from stgen.problem import make_problem, spatial_factors

pytestmark = pytest.mark.gpu

# (dim, cells, k): coarse orders 1572, 4484, 2806 (3d) and 8934
COARSE = {
    "2d_16x4_dg1": (2, (16, 4), 1),
    "2d_24x8_dg1": (2, (24, 8), 1),
    "3d_8x2x2_dg1": (3, (8, 2, 2), 1),
    "2d_32x8_dg2": (2, (32, 8), 2),
}
# real order 36004 of the time-decoupled block (2 n_s, n_s = 18002): past
# 256 tournament workgroups
LARGE = {"2d_80x20_dg1": (2, (80, 20), 1)}


@functools.lru_cache(maxsize=None)
def coarse_case(name):
    dim, n, k = {**COARSE, **LARGE}[name]
    p = make_problem(dim, n, 1, k, 0.01, 1e-3, 7)
    ol = oracle.prepare_levels(p.levels, p.b)
    J = ol[0].J.tocsc()
    lu = sla.splu(J)
    cond = sla.onenormest(J) * sla.onenormest(
        sla.LinearOperator(J.shape, matvec=lu.solve, rmatvec=lambda v: lu.solve(v, trans="T")))
    return p, J, lu, cond


@pytest.fixture(scope="module")
def stv():
    import paper_2107_10561_amd as m
    return m


def solve_on_gpu(stv, p, algo, r):
    s = stv.Solver(0)
    s.set_coarse_algorithm(algo)
    s.set_hierarchy(p.levels, p.dim, p.k)
    s.build_cell_inverses()
    d = to_dev(np.zeros_like(r))
    s.coarse_solve(to_dev(r), d)
    return to_host(d)


@pytest.mark.parametrize("name", list(COARSE))
def test_coarse_inverse_every_schedule(stv, name):
    p, J, lu, cond = coarse_case(name)
    r = np.random.default_rng(21).standard_normal(J.shape[0])
    ref = lu.solve(r)
    out = {}
    for algo in ("panels", "slabs", "tournament"):
        log(f"[coarse] {name} n={J.shape[0]} {algo}")
        d = solve_on_gpu(stv, p, algo, r)
        res = np.linalg.norm(r - J @ d) / np.linalg.norm(r)
        fe = relerr(d, ref)
        log(f"[coarse] {name} {algo} relres {res:.2e} forward {fe:.2e} cond {cond:.1e}")
        assert res <= 1e-11
        assert fe <= 1e-15 * cond * 10
        out[algo] = d
    # the same pivot sequence: the schedules differ only in rounding order
    assert relerr(out["panels"], out["slabs"]) <= 1e-15 * cond * 10


def solve_decoupled_on_gpu(stv, p, algo, r):
    """The coarse solve with the level's spatial factors set: the inverse is
    built from the real forms of the diagonal blocks T_p (x) M + I (x) A of
    the operator in the real Jordan basis of the time matrix (order 2 n_s
    each), eliminated with complex pivots by the tournament schedule."""
    _, w, C, _ = fe_time.time_matrices(p.k)
    s = stv.Solver(0)
    s.set_coarse_algorithm(algo)
    s.set_hierarchy(p.levels, p.dim, p.k)
    m, a = spatial_factors(p.levels[0])
    s.set_kron_factors(0, m, a, np.asarray(C, dtype=np.float64),
                       p.tau * np.asarray(w, dtype=np.float64))
    s.build_cell_inverses()
    d = to_dev(np.zeros_like(r))
    s.coarse_solve(to_dev(r), d)
    return to_host(d)


@pytest.mark.parametrize("name", list(COARSE))
def test_time_decoupled_coarse_inverse_every_schedule(stv, name):
    """Orders 2 n_s = 1572 (two workgroups of 128 complex rows, ragged),
    4484 and 2806 (merge trees of two levels), 5956 (slabs of 128): the same
    residual and forward-error bounds as the whole-matrix elimination, for
    the complex-pivot tournament and for the real schedules on the same real
    form."""
    p, J, lu, cond = coarse_case(name)
    r = np.random.default_rng(22).standard_normal(J.shape[0])
    ref = lu.solve(r)
    for algo in ("tournament", "slabs"):
        log(f"[coarse] {name} decoupled {algo}")
        d = solve_decoupled_on_gpu(stv, p, algo, r)
        res = np.linalg.norm(r - J @ d) / np.linalg.norm(r)
        fe = relerr(d, ref)
        log(f"[coarse] {name} decoupled {algo} relres {res:.2e} forward {fe:.2e} cond {cond:.1e}")
        assert res <= 1e-11
        assert fe <= 1e-15 * cond * 10


@pytest.mark.parametrize("name", list(LARGE))
def test_time_decoupled_coarse_two_level_merge_tree(stv, name):
    """Real order 36004 (padded to 36096): 282 tournament workgroups of 128
    real rows, so the complex tournament's merge tree takes two levels of
    16-list merges (282 -> 18 -> 2 lists for the root), the only case here
    past one level.  Complex tournament only (the real schedules' narrow
    panels would each sweep the 10 GB matrix); the same residual and
    forward-error bounds against SuperLU."""
    p, J, lu, cond = coarse_case(name)
    r = np.random.default_rng(26).standard_normal(J.shape[0])
    ref = lu.solve(r)
    log(f"[coarse] {name} decoupled tournament, order {J.shape[0]}")
    d = solve_decoupled_on_gpu(stv, p, "tournament", r)
    res = np.linalg.norm(r - J @ d) / np.linalg.norm(r)
    fe = relerr(d, ref)
    log(f"[coarse] {name} relres {res:.2e} forward {fe:.2e} cond {cond:.1e}")
    assert res <= 1e-11
    assert fe <= 1e-15 * cond * 10


@pytest.mark.parametrize("name", ["2d_16x4_dg1", "2d_32x8_dg2"])
@pytest.mark.parametrize("algo", ["tournament", "slabs", "panels"])
def test_time_decoupled_coarse_apply_both_directions(stv, name, algo):
    """The time-decoupled coarse inverse is applied from the eliminated blocks
    where the elimination left them: through paired pivot records (complex
    pivots, tournament) or real ones (slabs, panels), forward (coarse solve)
    and transposed (the V-cycle of the transposed one-level hierarchy is
    J^-T r).  dG(1): one complex pair; dG(2): a real eigenvalue and a pair."""
    p, J, lu, cond = coarse_case(name)
    _, w, C, _ = fe_time.time_matrices(p.k)
    s = stv.Solver(0)
    s.set_coarse_algorithm(algo)
    s.set_hierarchy(p.levels, p.dim, p.k)
    m, a = spatial_factors(p.levels[0])
    s.set_kron_factors(0, m, a, np.asarray(C, dtype=np.float64),
                       p.tau * np.asarray(w, dtype=np.float64))
    s.build_cell_inverses(full=True)
    r = np.random.default_rng(23).standard_normal(J.shape[0])
    for trans in (False, True):
        d = to_dev(np.zeros_like(r))
        if trans:
            s.vcycle_transposed(to_dev(r), d)
        else:
            s.coarse_solve(to_dev(r), d)
        d = to_host(d)
        A = J.T if trans else J
        ref = lu.solve(r, trans="T" if trans else "N")
        res = np.linalg.norm(r - A @ d) / np.linalg.norm(r)
        fe = relerr(d, ref)
        log(f"[coarse] {name} {algo} transposed={trans} relres {res:.2e} forward {fe:.2e}")
        assert res <= 1e-11
        assert fe <= 1e-15 * cond * 10
    s.close()


def test_coarse_algorithm_option_rejects_unknown(stv):
    s = stv.Solver(0)
    with pytest.raises(KeyError):
        s.set_coarse_algorithm("lu")
    with pytest.raises(stv.StvError):
        s._check(stv._lib.stv_set_option(s._h, 1, 7))


@pytest.mark.parametrize("singular", [False, True])
@pytest.mark.parametrize("name", ["2d_16x4_dg1", "2d_32x8_dg2", "3d_8x2x2_dg1", "2d_6x2_dg0"])
def test_coarse_solve_by_component(stv, name, singular):
    """With spatial factors and no prescribed schedule the coarse level is
    eliminated by velocity component and a pressure Schur complement.
    singular: one node's second component loses its velocity couplings, so its
    component block is singular although the coarse matrix is not; the build
    then eliminates the whole matrix.  Bounds as for the other schedules."""
    import scipy.sparse as sp
    dim, n, k = {**COARSE, "2d_6x2_dg0": (2, (6, 2), 0)}[name]
    p = make_problem(dim, n, 1, k, 0.01, 1e-3, 7)
    _, w, C, _ = fe_time.time_matrices(k)
    C, tw = np.asarray(C, dtype=np.float64), p.tau * np.asarray(w, dtype=np.float64)
    L = p.levels[0]
    m, a = (np.array(v) for v in spatial_factors(L))
    if singular:
        nv = 3 ** dim
        row = int(L.cell_sdofs[-1, nv + nv // 2])
        rows = np.repeat(np.arange(L.n_sdofs), np.diff(L.rowptr))
        hit = ((rows == row) | (np.asarray(L.col) == row)) & (m != 0.0)
        m[hit] = a[hit] = 0.0
        keep = int(np.nonzero((rows == row) & (np.asarray(L.col) == row))[0][0])
        a[keep] = 1e-300          # a stored diagonal, far below any other entry
    val = m[:, None, None] * C[None] + a[:, None, None] * np.diag(tw)[None]
    J = sp.bsr_matrix((val, L.col, L.rowptr), shape=(L.n_sdofs * p.b,) * 2).tocsc()
    lu = sla.splu(J)
    cond = sla.onenormest(J) * sla.onenormest(
        sla.LinearOperator(J.shape, matvec=lu.solve, rmatvec=lambda v: lu.solve(v, trans="T")))
    s = stv.Solver(0)
    s.set_hierarchy([dict(n_sdofs=L.n_sdofs, rowptr=L.rowptr, col=L.col, val=val,
                          cell_sdofs=L.cell_sdofs, P=None)], p.dim, p.k)
    s.set_kron_factors(0, m, a, C, tw)
    r = np.random.default_rng(28).standard_normal(J.shape[0])
    ref = lu.solve(r)
    for _ in range(2):
        s.build_cell_inverses()
        d = to_dev(np.zeros_like(r))
        s.coarse_solve(to_dev(r), d)
        d = to_host(d)
        res = np.linalg.norm(r - J @ d) / np.linalg.norm(r)
        fe = relerr(d, ref)
        log(f"[coarse] {name} singular={singular} relres {res:.2e} forward {fe:.2e} cond {cond:.1e}")
        assert res <= 1e-11 * max(1.0, 1e-8 * cond)
        assert fe <= 1e-15 * cond * 10


# kinds of coarse matrices given as blocks only: the velocity components apart,
# coupled (as in a Newton iteration), one node's velocity block singular, and a
# pressure block on the diagonal (eliminated as a whole)
@pytest.mark.parametrize("kind", ["apart", "coupled", "singular", "pressure"])
@pytest.mark.parametrize("case", [(2, [(16, 4)], 1), (3, [(8, 2, 2)], 1), (2, [(18, 2)], 0),
                                  (2, [(15, 3)], 2), (2, [(16, 4), (20, 2), (5, 3)], 1)])
def test_coarse_solve_of_blocks_by_separators(stv, case, kind):
    """Without spatial factors the coarse blocks are one real matrix, cut by
    separators and reduced to the border.  Bounds as for the other schedules."""
    import scipy.sparse as sp
    dim, shapes, k = case
    rng = np.random.default_rng(31)
    hier, mats = [], []
    for n in shapes:
        p = make_problem(dim, n, 1, k, 0.01, 1e-3, 7)
        L = p.levels[0]
        val = np.array(L.val)
        rows = np.repeat(np.arange(L.n_sdofs), np.diff(L.rowptr))
        col = np.asarray(L.col)
        nv = 3 ** dim
        comp = np.full(L.n_sdofs, dim)
        for d in range(dim):
            comp[np.asarray(L.cell_sdofs)[:, d * nv:(d + 1) * nv]] = d
        if kind == "coupled":
            hit = (comp[rows] < dim) & (comp[col] < dim) & (comp[rows] != comp[col])
            scale = 1e-2 * np.median(np.abs(val[(rows == col) & (comp[rows] == 0)]).max(axis=(1, 2)))
            val[hit] = scale * rng.uniform(-1, 1, (int(hit.sum()), p.b, p.b))
        elif kind == "singular":
            row = int(L.cell_sdofs[-1, nv + nv // 2])
            hit = ((rows == row) | (col == row)) & (comp[rows] < dim) & (comp[col] < dim)
            val[hit] = 0.0
            val[(rows == row) & (col == row)] = 1e-300 * np.eye(p.b)
        elif kind == "pressure":
            hit = (rows == col) & (comp[rows] == dim)
            val[hit] = 1e-3 * np.abs(val).max() * np.eye(p.b)
        hier.append([dict(n_sdofs=L.n_sdofs, rowptr=L.rowptr, col=L.col, val=val,
                          cell_sdofs=L.cell_sdofs, P=None)])
        mats.append(sp.bsr_matrix((val, L.col, L.rowptr), shape=(L.n_sdofs * p.b,) * 2).tocsc())
    s = stv.Solver(0)
    s.set_batch(hier, dim, k) if len(hier) > 1 else s.set_hierarchy(hier[0], dim, k)
    r = rng.standard_normal(sum(J.shape[0] for J in mats))
    for _ in range(2):
        s.build_cell_inverses()
        dd = to_dev(np.zeros_like(r))
        s.coarse_solve(to_dev(r), dd)
        d, at = to_host(dd), 0
        for n, J in zip(shapes, mats):
            sl = slice(at, at + J.shape[0])
            at += J.shape[0]
            lu = sla.splu(J)
            cond = sla.onenormest(J) * sla.onenormest(
                sla.LinearOperator(J.shape, matvec=lu.solve, rmatvec=lambda v: lu.solve(v, trans="T")))
            res = np.linalg.norm(r[sl] - J @ d[sl]) / np.linalg.norm(r[sl])
            fe = relerr(d[sl], lu.solve(r[sl]))
            log(f"[coarse] blocks {dim}d {n} k={k} {kind} relres {res:.2e} forward {fe:.2e} cond {cond:.1e}")
            assert res <= 1e-11 * max(1.0, 1e-8 * cond)
            assert fe <= 1e-15 * cond * 10
    s.close()


@pytest.mark.parametrize("factors", [False, True])
@pytest.mark.parametrize("case", [(2, (4, 1), 1), (2, (16, 4), 0), (2, (16, 4), 1), (2, (9, 3), 2),
                                  (2, (8, 3), 3), (3, (4, 2, 2), 1)])
@pytest.mark.parametrize("full", [False, True])
def test_whole_inverse_from_parts(stv, case, factors, full):
    """The whole coarse inverse made of the parts' inverses and the border's
    (all time blocks recombined): forward, and transposed with the all-rows
    layout.  Bounds as for the other schedules."""
    dim, n, k = case
    p = make_problem(dim, n, 1, k, 0.01, 1e-3, 7)
    J = oracle.prepare_levels(p.levels, p.b)[0].J.tocsc()
    lu = sla.splu(J)
    cond = sla.onenormest(J) * sla.onenormest(
        sla.LinearOperator(J.shape, matvec=lu.solve, rmatvec=lambda v: lu.solve(v, trans="T")))
    s = stv.Solver(0)
    s.set_hierarchy(p.levels, dim, k)
    if factors:
        _, w, C, _ = fe_time.time_matrices(k)
        m, a = spatial_factors(p.levels[0])
        s.set_kron_factors(0, m, a, np.asarray(C, dtype=np.float64),
                           p.tau * np.asarray(w, dtype=np.float64))
    s.build_cell_inverses(full=full)
    r = np.random.default_rng(37).standard_normal(J.shape[0])
    for trans in ((False, True) if full else (False,)):
        dd = to_dev(np.zeros_like(r))
        s.vcycle_transposed(to_dev(r), dd) if trans else s.coarse_solve(to_dev(r), dd)
        d, A = to_host(dd), J.T if trans else J
        res = np.linalg.norm(r - A @ d) / np.linalg.norm(r)
        fe = relerr(d, lu.solve(r, trans="T" if trans else "N"))
        log(f"[coarse] whole {case} factors={factors} full={full} transposed={trans} "
            f"relres {res:.2e} forward {fe:.2e} cond {cond:.1e}")
        assert res <= 1e-11 * max(1.0, 1e-8 * cond)
        assert fe <= 1e-15 * cond * 10
    s.close()
