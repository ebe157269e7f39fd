"""Cell inverses and sweeps of levels whose velocity components do not couple
(one elimination per distinct component block and a pressure Schur complement):
against the oracle, which inverts each whole J_T; and an operator with a cell
whose component block is singular although J_T is not, which the build has to
eliminate as a whole."""
import numpy as np
import pytest

import oracle
from gpu_common import relerr, to_dev, to_host
from stgen import fe
from stgen.problem import make_problem, spatial_factors

pytestmark = pytest.mark.gpu

# (dim, finest cells, levels, k): 2d real block + pair and pair alone, 3d pair
# with every kind of wall cell (27 to 8 owned nodes: both row tiles of the sweep)
CASES = {"2d_dg1": (2, (10, 6), 2, 1), "2d_dg2": (2, (12, 4), 2, 2), "3d_dg1": (3, (6, 4, 2), 2, 1),
         "3d_dg1_interior": (3, (4, 4, 6), 2, 1)}


@pytest.fixture(scope="module")
def stv():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    import paper_2107_10561_amd as m
    return m


def _system(name, singular):
    dim, n, G, k = CASES[name]
    p = make_problem(dim, n, G, k, 0.01, 1e-3, 17)
    _, w, C, _ = fe.time_matrices(k)
    C, tw = np.asarray(C, dtype=np.float64), p.tau * np.asarray(w, dtype=np.float64)
    levels, factors = [], []
    for g, L in enumerate(p.levels):
        m, a = (np.array(v) for v in spatial_factors(L))
        if singular and g == G - 1:
            # the second component at the centre node of the last cell: no
            # velocity couplings left, only those with the pressure
            nv = 3 ** dim
            s = int(L.cell_sdofs[-1, nv + nv // 2])
            rows = np.repeat(np.arange(L.n_sdofs), np.diff(L.rowptr))
            hit = ((rows == s) | (np.asarray(L.col) == s)) & (m != 0.0)
            m[hit] = a[hit] = 0.0
        val = m[:, None, None] * C[None] + a[:, None, None] * np.diag(tw)[None]
        levels.append(dict(n_sdofs=L.n_sdofs, rowptr=L.rowptr, col=L.col, val=val,
                           cell_sdofs=L.cell_sdofs, P=L.P))
        factors.append((m, a))
    return p, levels, factors, C, tw


@pytest.mark.parametrize("singular", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_component_cells(stv, name, singular):
    p, levels, factors, C, tw = _system(name, singular)
    ol = oracle.build_inverses(oracle.prepare_levels(levels, p.b))
    g, L = len(levels) - 1, levels[-1]
    own = oracle.owner_cells(L["cell_sdofs"], L["n_sdofs"])
    nls = L["cell_sdofs"].shape[1]
    # an inverse is good to about cond(J_T) roundings per accumulated term
    cond = max(np.linalg.norm(oracle.extract_cell_matrix(ol[g].J, ol[g].dofs[T]), 2) *
               np.linalg.norm(ol[g].inv[T], 2) for T in (0, len(ol[g].inv) - 1))
    tol = max(1e-12, 64 * 2.0 ** -53 * cond)
    rng = np.random.default_rng(5)
    r, d0 = rng.standard_normal(ol[g].n_st), rng.standard_normal(ol[g].n_st)
    r *= np.abs(ol[g].J @ d0).max()
    ref = oracle.vanka_sweep(ol[g], r, oracle.vanka_sweep(ol[g], r, d0, 0.7), 0.7)
    for fp32 in (False, True):
        s = stv.Solver(0)
        s.set_hierarchy(levels, p.dim, p.k)
        for lv, (m, a) in enumerate(factors):
            s.set_kron_factors(lv, m, a, C, tw)
        s.build_cell_inverses(fp32=fp32)
        s.build_cell_inverses(fp32=fp32)   # a second build in place
        if not fp32:
            for T in range(L["cell_sdofs"].shape[0]):
                O, G = ol[g].inv[T], s.get_cell_inverse(g, T)
                rows = [l * nls + a for l in range(p.b) for a in range(nls)
                        if own[L["cell_sdofs"][T, a]] == T]
                assert np.abs(G[rows] - O[rows]).max() <= tol * np.abs(O).max(), T
        for wgs in (0, 1, 3):
            s.set_launch(g, 2, wgs)
            d = to_dev(d0)
            s.vanka_sweep(g, to_dev(r), d, 2, 0.7)
            # FP32 store: 2^-24 per value, times the inverse's condition at most
            assert relerr(to_host(d), ref) <= (max(1e-5, 2.0 ** -24 * cond) if fp32 else tol), wgs


@pytest.mark.parametrize("cells", [(56, 2, 2), (38, 6, 2), (56, 4, 2), (30, 4, 4)])
@pytest.mark.parametrize("k", [1, 2])
def test_block_cells_in_chunks(stv, cells, k):
    """3d cells without factors, built beside the coarse chain in launches of
    7/8 of the compute units (224 of 256): 224, 456, 448 and 480 cells; first,
    last and the cells on both sides of every cut, against the oracle."""
    p = make_problem(3, cells, 2, k, 0.01, 1e-3, 17)
    L = p.levels[-1]
    own = oracle.owner_cells(L.cell_sdofs, L.n_sdofs)
    nls, n = L.cell_sdofs.shape[1], L.cell_sdofs.shape[0]
    s = stv.Solver(0)
    s.set_hierarchy(p.levels, 3, k)
    s.build_cell_inverses()
    for T in sorted({0, 223, 224 % n, 447 % n, 448 % n, n - 1}):
        JT = oracle.extract_cell_matrix_blocks(L.rowptr, L.col, L.val, p.b, L.cell_sdofs[T])
        O, G = oracle.cell_inverse(JT), s.get_cell_inverse(1, T)
        rows = [l * nls + a for l in range(p.b) for a in range(nls)
                if own[L.cell_sdofs[T, a]] == T]
        tol = max(1e-12, 64 * 2.0 ** -53 * np.linalg.norm(JT, 2) * np.linalg.norm(O, 2))
        assert np.abs(G[rows] - O[rows]).max() <= tol * np.abs(O).max(), T
    s.close()
