"""Set-up of a hierarchy: the threaded index checks name the lowest bad row and
cell, and the level operators are whole on the device whichever way they were
sent (one copy per array, or the pinned ring above 8 MB; one member or two)."""
import numpy as np
import pytest

from stgen.problem import make_problem


@pytest.fixture(scope="module")
def stv():
    import paper_2107_10561_amd as m
    return m


def _levels(n, levels, k=1):
    p = make_problem(2, n, levels, k, 0.01, 1e-3, 23)
    return p, [dict(n_sdofs=L.n_sdofs, rowptr=np.array(L.rowptr, dtype=np.int32),
                    col=np.array(L.col), val=L.val, cell_sdofs=np.array(L.cell_sdofs),
                    P=L.P) for L in p.levels]


# bad rows in the first, a middle and the last thread's range; two at once
@pytest.mark.parametrize("rows", [[0], [70001], [-1], [-1, 20000]])
def test_lowest_bad_row_and_cell(stv, rows):
    _, lv = _levels((192, 96), 2)
    L = lv[-1]
    assert stv.validate_hierarchy(lv, 2, 1)[0] == stv.STV_OK
    rows = [r % L["n_sdofs"] for r in rows]
    for r in rows:
        q = L["rowptr"][r]
        L["col"][q], L["col"][q + 1] = L["col"][q + 1], L["col"][q]
    rc, msg = stv.validate_hierarchy(lv, 2, 1)
    assert rc == stv.STV_EINVAL
    assert f"strictly increasing per row (row {min(rows)})" in msg, msg
    for r in rows:
        q = L["rowptr"][r]
        L["col"][q], L["col"][q + 1] = L["col"][q + 1], L["col"][q]
    cells = [r % len(L["cell_sdofs"]) for r in rows]
    for c in cells:   # the last velocity DoF twice
        L["cell_sdofs"][c, 17] = L["cell_sdofs"][c, 16]
    rc, msg = stv.validate_hierarchy(lv, 2, 1)
    assert rc == stv.STV_EINVAL and f"repeated DoF in cell {min(cells)}" in msg, msg


# values of 1.5 MB (copies) to 81 MB a member (ring; no multiple of its chunk)
@pytest.mark.gpu
@pytest.mark.parametrize("n", [(24, 8), (48, 22), (128, 41), (192, 56)])
@pytest.mark.parametrize("members", [1, 2])
def test_operators_arrive_whole(stv, n, members):
    import torch
    s = stv.Solver()
    p, lv = _levels(n, 1)
    if members == 1:
        s.set_hierarchy(lv, 2, 1)
    else:
        s.set_batch([lv] * members, 2, 1)
    L, b = lv[0], p.b
    n_s = L["n_sdofs"]
    d = np.random.default_rng(5).standard_normal((members, n_s, b))
    rows = np.repeat(np.arange(n_s), np.diff(L["rowptr"]))
    want = np.zeros_like(d)
    scale = np.zeros_like(d)
    for i in range(members):
        x = d[i][L["col"]]
        np.add.at(want[i], rows, -np.einsum("nij,nj->ni", L["val"], x))
        np.add.at(scale[i], rows, np.einsum("nij,nj->ni", np.abs(L["val"]), np.abs(x)))
    dd = torch.from_numpy(d.reshape(-1)).cuda()
    zero = torch.zeros_like(dd)
    out = torch.empty_like(dd)
    s.residual(0, zero, dd, out)
    got = out.cpu().numpy().reshape(want.shape)
    # sums of at most some 200 products in two orders
    assert np.all(np.abs(got - want) <= 400 * np.finfo(float).eps * scale + 1e-300)
