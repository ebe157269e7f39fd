"""Cell problems whose velocity block is nearly singular although the cell's
matrix is not: eliminated by component or as a whole, the stored inverse is the
oracle's to the rounding of a pivoted inverse."""
import numpy as np
import pytest

import oracle
from gpu_common import log
from stgen import fe
from stgen.problem import make_problem, spatial_factors

pytestmark = pytest.mark.gpu

# 2d: one pair; a real block and a pair; 3d: one pair
CASES = {"2d_dg1": (2, (10, 6), 1), "2d_dg2": (2, (12, 4), 2), "3d_dg1": (3, (4, 4, 2), 1)}


@pytest.mark.parametrize("delta", [1e-1, 1e-3, 1e-5, 1e-6, 2e-7])
@pytest.mark.parametrize("kind", ["node", "row"])
@pytest.mark.parametrize("name", list(CASES))
def test_weak_velocity_node(name, kind, delta):
    """The velocity couplings of one node of the last cell (its centre, second
    component) scaled to delta of the block: node = a diagonal entry alone,
    row = its whole row.  Tolerance: the build accepts cancellations of up to
    4096 roundings, and 8 roundings per unit of condition otherwise."""
    import paper_2107_10561_amd as stv
    dim, n, k = CASES[name]
    p = make_problem(dim, n, 2, k, 0.01, 1e-3, 17)
    _, w, C, _ = fe.time_matrices(k)
    C, tw = np.asarray(C, dtype=np.float64), p.tau * np.asarray(w, dtype=np.float64)
    levels, factors = [], []
    for g, L in enumerate(p.levels):
        m, a = (np.array(v) for v in spatial_factors(L))
        if g == 1:
            nv = 3 ** dim
            s = int(L.cell_sdofs[-1, nv + nv // 2])
            rows, col = np.repeat(np.arange(L.n_sdofs), np.diff(L.rowptr)), np.asarray(L.col)
            vel = np.zeros(L.n_sdofs, dtype=bool)
            vel[np.asarray(L.cell_sdofs)[:, :dim * nv]] = True
            diag = (rows == s) & (col == s)
            if kind == "node":
                md, ad = m[diag][0], a[diag][0]
                hit = ((rows == s) | (col == s)) & vel[rows] & vel[col]
                m[hit] = a[hit] = 0.0
                m[diag], a[diag] = delta * md, delta * ad
            else:
                hit = (rows == s) & vel[col]
                m[hit] *= delta
                a[hit] *= delta
        levels.append(dict(n_sdofs=L.n_sdofs, rowptr=L.rowptr, col=L.col,
                           val=m[:, None, None] * C[None] + a[:, None, None] * np.diag(tw)[None],
                           cell_sdofs=L.cell_sdofs, P=L.P))
        factors.append((m, a))
    L = levels[1]
    own = oracle.owner_cells(L["cell_sdofs"], L["n_sdofs"])
    nls = L["cell_sdofs"].shape[1]
    s = stv.Solver(0)
    s.set_hierarchy(levels, dim, k)
    for g, (m, a) in enumerate(factors):
        s.set_kron_factors(g, m, a, C, tw)
    s.build_cell_inverses()
    worst = 0.0
    for T in range(len(L["cell_sdofs"])):
        JT = oracle.extract_cell_matrix_blocks(L["rowptr"], L["col"], L["val"], p.b, L["cell_sdofs"][T])
        O, G = oracle.cell_inverse(JT), s.get_cell_inverse(1, T)
        rows = [l * nls + a for l in range(p.b) for a in range(nls) if own[L["cell_sdofs"][T, a]] == T]
        if not rows:
            continue
        cond = np.linalg.norm(JT, 2) * np.linalg.norm(O, 2)
        err = np.abs(G[rows] - O[rows]).max() / np.abs(O).max()
        worst = max(worst, err / max(4096.0, 8.0 * cond))
        assert err <= 2.0 ** -53 * max(4096.0, 8.0 * cond), (T, err, cond)
    log(f"[cells] {name} {kind} {delta:g} worst {worst / 2.0 ** -53:.2f} of the bound")
    s.close()
