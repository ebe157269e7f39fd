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


@pytest.mark.parametrize("fp32", [False, True])
def test_nodes_owned_in_some_components(fp32):
    """A node whose third component is another DoF in the last cell: the cell
    before owns that component alone, the last one the others and the new DoF
    (3d component store).  Two sweeps against the oracle, 2^-24 per value of an
    FP32 store times the condition at most."""
    import scipy.sparse as sp
    import paper_2107_10561_amd as stv
    from gpu_common import relerr, to_dev, to_host
    p = make_problem(3, (4, 4, 2), 2, 1, 0.01, 1e-3, 17)
    _, w, C, _ = fe.time_matrices(1)
    C, tw = np.asarray(C, dtype=np.float64), p.tau * np.asarray(w, dtype=np.float64)
    levels, factors = [], []
    for g, L in enumerate(p.levels):
        m, a = (np.array(v) for v in spatial_factors(L))
        n, csd, P = L.n_sdofs, np.array(L.cell_sdofs), L.P
        rowptr, col = np.asarray(L.rowptr), np.asarray(L.col)
        if g == 1:
            # node of the last cell that the cell before shares, third component
            j = next(j for j in range(27) if csd[-1, 54 + j] in csd[-2] and j != 13)
            old = csd[-1, 54 + j]
            csd[-1, 54 + j] = n
            q = np.arange(rowptr[old], rowptr[old + 1])
            order = np.argsort(np.where(col[q] == old, n, col[q]))
            col = np.concatenate([col, np.where(col[q] == old, n, col[q])[order]]).astype(col.dtype)
            m, a = np.concatenate([m, m[q][order]]), np.concatenate([a, a[q][order]])
            rowptr = np.concatenate([rowptr, [rowptr[-1] + len(q)]]).astype(rowptr.dtype)
            pr, pc, pv = P
            k = np.arange(pr[old], pr[old + 1])
            P = (np.concatenate([pr, [pr[-1] + len(k)]]).astype(pr.dtype), np.concatenate([pc, pc[k]]),
                 np.concatenate([pv, pv[k]]))
            n += 1
        levels.append(dict(n_sdofs=n, rowptr=rowptr, col=col,
                           val=m[:, None, None] * C[None] + a[:, None, None] * np.diag(tw)[None],
                           cell_sdofs=csd, P=P))
        factors.append((m, a))
    own = oracle.owner_cells(levels[1]["cell_sdofs"], levels[1]["n_sdofs"])
    assert own[old] != len(levels[1]["cell_sdofs"]) - 1 and own[-1] == len(levels[1]["cell_sdofs"]) - 1
    ol = oracle.build_inverses(oracle.prepare_levels(levels, 2))
    rng = np.random.default_rng(7)
    r, d0 = rng.standard_normal(ol[1].n_st), rng.standard_normal(ol[1].n_st)
    r *= np.abs(ol[1].J @ d0).max()
    ref = oracle.vanka_sweep(ol[1], r, oracle.vanka_sweep(ol[1], r, d0, 0.7), 0.7)
    cond = max(np.linalg.norm(oracle.extract_cell_matrix(ol[1].J, ol[1].dofs[T]), 2) *
               np.linalg.norm(ol[1].inv[T], 2) for T in (0, len(ol[1].inv) - 1))
    s = stv.Solver(0)
    s.set_hierarchy(levels, 3, 1)
    for g, (m, a) in enumerate(factors):
        s.set_kron_factors(g, m, a, C, tw)
    s.build_cell_inverses(fp32=fp32)
    d = to_dev(d0)
    s.vanka_sweep(1, to_dev(r), d, 2, 0.7)
    err = relerr(to_host(d), ref)
    log(f"[cells] nodes owned in part fp32={fp32} err {err:.1e} cond {cond:.1e}")
    assert err <= (2.0 ** -24 * cond if fp32 else 2.0 ** -53 * max(4096.0, 8.0 * cond))
    s.close()
