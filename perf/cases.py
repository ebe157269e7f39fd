"""Performance cases of the space-time Vanka multigrid.

Each case is one call, or one short sequence of calls, that a program using
the solver makes on the device, on a channel problem of the given mesh (`nx`,
`ny`, `nz` finest cells, `levels` levels by uniform coarsening, dG(`k`) in
time).  Kinds:

  step      cell and coarse inverses, then FGMRES: one implicit time step of
            the Oseen system with the spatial factors known to the solver
  batch     the same for many independent 2d problems of uneven size at once
  newton    set_hierarchy + inverses + FGMRES for a Jacobian whose time blocks
            are full (no spatial factors): one step of a Newton iteration,
            where every step brings new values
  blocks    inverses + FGMRES for such a Jacobian on the resident hierarchy
  gradient  inverses with all rows, forward and transposed FGMRES and the
            gradient of every cell's viscosity
  vcycle    one V(2,2) cycle, as a preconditioner inside another Krylov method
  smooth    two Vanka sweeps on the finest level
  residual  r - J d on the finest level

FGMRES runs a fixed number of steps (about what relative residual 1e-8 takes
on these problems), so that every run does the same work.  The operator of a
seed differs from another's by the time step (in a batch by the viscosity of
each problem, for the gradient by the viscosity of each cell); right-hand sides
are N(0, 1).
"""
from __future__ import annotations

import functools
import random

import numpy as np
import torch

import paper_2107_10561_amd as stv
from stgen import adjoint, fe, newton
from stgen.assemble import assemble_spatial_factors, bsr_pattern
from stgen.mesh import Mesh, prolongation
from stgen.problem import H2D, H3D, L2D, L3D, Convection

DEV = "cuda:0"
NU = 1e-3
OMEGA = 0.7
KINDS = ("step", "batch", "newton", "blocks", "gradient", "vcycle", "smooth", "residual")
# finest meshes and levels of the problems a batch draws from
BATCH_MESHES = (((32, 8), 3), ((64, 16), 4), ((96, 24), 4), ((128, 32), 5))


def _case(kind, mesh, levels, k, fp32=False, iters=0, **more):
    nx, ny, nz = (*mesh, 0)[:3]
    return dict(kind=kind, nx=nx, ny=ny, nz=nz, levels=levels, k=k, fp32=fp32, iters=iters, **more)


def listed():
    cases = {
        # the smallest problem the solver is used on: latency and launches
        "step_2d_16x4_dg1": _case("step", (16, 4), 2, 1, iters=11),
        # one ordinary 2d problem, FP32-stored inverses
        "step_2d_128x32_dg1_fp32": _case("step", (128, 32), 5, 1, True, 11),
        # the large 2d channel with three time components
        "step_2d_512x128_dg2": _case("step", (512, 128), 6, 2, iters=11),
        # an ordinary 3d problem, FP32-stored inverses
        "step_3d_48x12x12_dg1_fp32": _case("step", (48, 12, 12), 3, 1, True, 10),
        # the largest 3d channel
        "step_3d_128x24x24_dg1": _case("step", (128, 24, 24), 4, 1, iters=10),
        # many uneven problems at once (ensembles, parameter studies)
        "batch_64_2d_dg1_fp32": dict(kind="batch", n=64, k=1, fp32=True, iters=11),
        # one Newton step of a 2d time march, upload of the Jacobian included
        "newton_2d_256x64_dg1": _case("newton", (256, 64), 5, 1, iters=9),
        # a 3d Jacobian with full time blocks
        "blocks_3d_32x8x8_dg1": _case("blocks", (32, 8, 8), 3, 1, iters=10),
        # gradient of an outflow loss by the adjoint solve
        "gradient_2d_256x64_dg1": _case("gradient", (256, 64), 5, 1, iters=8),
        # the preconditioner alone, odd coarse mesh, lowest time order
        "vcycle_2d_200x56_dg0": _case("vcycle", (200, 56), 4, 0),
        # the smoother alone, 3d, odd coarse mesh
        "smooth_3d_40x20x12_dg1": _case("smooth", (40, 20, 12), 3, 1),
        # the residual alone, 2d, between the two 2d steps in size
        "residual_2d_336x80_dg2": _case("residual", (336, 80), 4, 2),
    }
    return [dict(c, name=name) for name, c in cases.items()]


def draw(rng: random.Random):
    kind = rng.choice(KINDS)
    if kind == "batch":
        return dict(kind=kind, n=round(2 ** rng.uniform(1, 6)), k=1, fp32=rng.random() < 0.7,
                    iters=rng.randint(8, 11))
    iters = 0 if kind in ("vcycle", "smooth", "residual") else rng.randint(7, 12)
    fp32 = kind in ("step", "blocks", "newton") and rng.random() < 0.4
    three_d = kind in ("step", "vcycle", "smooth", "residual", "blocks") and rng.random() < 0.5
    # the general blocks are larger per cell and assembled anew for each seed
    small = kind in ("newton", "blocks", "gradient")
    top = (2048 if small else 73728) if three_d else (16384 if small else 65536)
    target = 2 ** rng.uniform(6, np.log2(top))
    while True:
        levels = rng.randint(2, 4 if three_d else 6)
        f = 2 ** (levels - 1)
        coarse = (rng.randint(2, 16), rng.randint(1, 3), rng.randint(1, 3)) if three_d else \
            (rng.randint(4, 20), rng.randint(1, 6))
        cells = int(np.prod([c * f for c in coarse]))
        if cells <= top and target / 2 <= cells <= target * 2:
            break
    k = 1 if kind == "gradient" else rng.randint(0, 1 if three_d else 2)
    if kind in ("newton", "blocks"):
        k = max(k, 1)
    return _case(kind, tuple(c * f for c in coarse), levels, k, fp32, iters)


# ------------------------------------------------------------------ problems
class _Geometry:
    """Meshes, patterns, transfers and spatial operators of one hierarchy,
    coarsest level first; assembled once per mesh, as a program that marches
    in time does."""

    def __init__(self, n, levels):
        dim = len(n)
        ext = (L2D, H2D) if dim == 2 else (L3D, H3D, H3D)
        meshes = [Mesh(dim, tuple(n), ext)]
        for _ in range(levels - 1):
            meshes.append(meshes[-1].coarsen())
        self.dim, self.meshes = dim, meshes[::-1]
        self.csd = [m.cell_sdofs() for m in self.meshes]
        self.P = [None] + [prolongation(self.meshes[g], self.meshes[g - 1])
                           for g in range(1, levels)]
        self.pattern = [bsr_pattern(m, c) for m, c in zip(self.meshes, self.csd)]
        amps = np.random.default_rng(1001).standard_normal((4,) if dim == 2 else (4, 3))
        self.conv = Convection(dim, ext, amps).normalise()

    def factors(self, nu, conv):
        return [assemble_spatial_factors(m, np.full(m.n_cells, nu), conv, *self.pattern[g])
                for g, m in enumerate(self.meshes)]

    @functools.cached_property
    def oseen(self):
        """(M, A) per level at viscosity NU."""
        return self.factors(NU, self.conv)

    @functools.cached_property
    def split(self):
        """(M, rest, viscous, convective) per level: A = rest + nu viscous + convective."""
        def still(x):
            return np.zeros_like(x)
        parts = zip(self.factors(0.0, still), self.factors(1.0, still), self.factors(0.0, self.conv))
        return [(m, a0, a1 - a0, ac - a0) for (m, a0), (_, a1), (_, ac) in parts]

    def level(self, g, val):
        rowptr, col = self.pattern[g]
        return dict(n_sdofs=self.meshes[g].n_sdofs, rowptr=rowptr, col=col, val=val,
                    cell_sdofs=self.csd[g], P=self.P[g])


@functools.lru_cache(maxsize=4)
def _geometry(n, levels):
    return _Geometry(n, levels)


def _mesh(case):
    return tuple(case[a] for a in ("nx", "ny", "nz") if case[a])


def _tau(k, seed):
    """The seed's time step, around 0.01 (0.005 for dG(2))."""
    return (0.005 if k == 2 else 0.01) * (0.8 + 0.4 * random.Random(seed).random())


def _time(k, tau):
    _, w, C, _ = fe.time_matrices(k)
    return np.asarray(C, dtype=np.float64), tau * np.asarray(w, dtype=np.float64)


def _kron_blocks(m, a, C, tw):
    """Block values C (x) m + diag(tw) (x) a, one (k+1) x (k+1) block per pair."""
    b = len(tw)
    m, a = torch.from_numpy(m), torch.from_numpy(a)
    val = torch.empty((m.numel(), b, b), dtype=torch.float64)
    for i in range(b):
        for l in range(b):
            torch.mul(m, float(C[i, l]), out=val[:, i, l])
        val[:, i, i].add_(a, alpha=float(tw[i]))
    return val.numpy()


def _oseen_levels(geo, k, tau):
    C, tw = _time(k, tau)
    return [geo.level(g, _kron_blocks(m, a, C, tw)) for g, (m, a) in enumerate(geo.oseen)]


def _full_levels(geo, k, tau):
    """The convection field varies linearly in time, so the time blocks of the
    Jacobian are full: C m + diag(tw) (rest + nu visc) + tau T.s conv."""
    C, tw = _time(k, tau)
    nodes = np.asarray(fe.time_matrices(k)[0], dtype=np.float64)
    S = tau * newton.time_triple(k) @ (1.0 + 0.5 * nodes)
    out = []
    for g, (m, rest, visc, conv) in enumerate(geo.split):
        val = _kron_blocks(m, rest + NU * visc, C, tw)
        val += conv[:, None, None] * S[None]
        out.append(geo.level(g, val))
    return out


def _randn(n, seed, stream=0):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(2 * seed + stream)
    return torch.randn(n, generator=gen, device=DEV, dtype=torch.float64)


def _pair(geo, k, tau, n, seed):
    """(r, d) with r about as large as J d, as they are inside a solve."""
    C, tw = _time(k, tau)
    m, a = geo.oseen[-1]
    scale = np.linalg.norm(C[0, 0] * m + tw[0] * a) / np.sqrt(geo.meshes[-1].n_sdofs)
    return _randn(n, seed) * scale, _randn(n, seed, 1)


def _factored_solver(levels, geo, k, tau, fp32):
    """A solver with the spatial factors set and its launch shapes tuned."""
    s = stv.Solver(0)
    s.set_hierarchy(levels, geo.dim, k)
    for g, (m, a) in enumerate(geo.oseen):
        s.set_kron_factors(g, m, a, *_time(k, tau))
    s.build_cell_inverses(fp32=fp32)
    s.autotune()
    return s


# ------------------------------------------------------------------ prepare
def prepare(case, seed):
    kind, k = case["kind"], case["k"]
    st = dict(kind=kind, fp32=case["fp32"], iters=case["iters"])
    if kind == "batch":
        return _prepare_batch(case, seed, st)
    if kind == "gradient":
        return _prepare_gradient(case, seed, st)
    geo = _geometry(_mesh(case), case["levels"])
    tau = _tau(k, seed)
    n = geo.meshes[-1].n_sdofs * (k + 1)
    st["rhs"] = _randn(n, seed)
    if kind in ("newton", "blocks"):
        levels = _full_levels(geo, k, tau)
        s = stv.Solver(0)
        s.set_hierarchy(levels, geo.dim, k)
        if kind == "newton":
            st.update(levels=levels, dim=geo.dim, k=k)
    else:
        s = _factored_solver(_oseen_levels(geo, k, tau), geo, k, tau, case["fp32"])
    st.update(solver=s, x=torch.zeros(n, dtype=torch.float64, device=DEV), top=case["levels"] - 1)
    if kind in ("smooth", "residual"):
        st["rhs"], st["d0"] = _pair(geo, k, tau, n, seed)
    return st


@functools.lru_cache(maxsize=2)
def _batch_choice(n):
    return [random.Random(2000 + j).choice(BATCH_MESHES) for j in range(n)]


def _prepare_batch(case, seed, st):
    k, tau = case["k"], 0.01
    C, tw = _time(k, tau)
    rng = random.Random(seed)
    members = []
    for n, levels in _batch_choice(case["n"]):
        geo = _geometry(n, levels)
        nu = rng.uniform(5e-4, 5e-3)
        members.append((geo, [(m, rest + nu * visc + conv) for m, rest, visc, conv in geo.split]))
    s = stv.Solver(0)
    s.set_batch([[geo.level(g, _kron_blocks(m, a, C, tw)) for g, (m, a) in enumerate(ma)]
                 for geo, ma in members], 2, k)
    for g in range(s.n_levels):
        # the packed level's members, aligned at the finest level
        here = [ma[g - s.n_levels + len(ma)] for _, ma in members if g >= s.n_levels - len(ma)]
        s.set_kron_factors(g, np.concatenate([m for m, _ in here]),
                           np.concatenate([a for _, a in here]), C, tw)
    s.build_cell_inverses(fp32=case["fp32"])
    s.autotune()
    n = s.n_st[-1]
    st.update(solver=s, rhs=_randn(n, seed), x=torch.zeros(n, dtype=torch.float64, device=DEV))
    return st


def _prepare_gradient(case, seed, st):
    k, tau = case["k"], 0.01
    p = adjoint.make_differentiation_problem(_mesh(case), case["levels"], k, tau, seed)
    fine = p.levels[-1].mesh
    refs, kptr, kidx, kw = adjoint.nu_derivative_refs(fine)
    F0, cells, Fc = adjoint.inflow_rhs_parts(fine, k, tau)
    s = stv.Solver(0)
    s.set_hierarchy(p.levels, p.dim, k)
    b = torch.from_numpy(p.rhs).to(DEV)
    st.update(solver=s, top=case["levels"] - 1, rhs=b, q=torch.from_numpy(p.loss).to(DEV),
              x=torch.zeros_like(b), lam=torch.zeros_like(b),
              grad=torch.zeros(fine.n_cells, dtype=torch.float64, device=DEV),
              terms=(refs, kptr, kidx, kw, adjoint.time_weights(k, tau)), cells=cells,
              f=np.ascontiguousarray(Fc.reshape(len(cells), -1)))
    return st


# ---------------------------------------------------------------------- run
def run(st):
    s, kind = st["solver"], st["kind"]
    if kind == "residual":
        s.residual(st["top"], st["rhs"], st["d0"], st["x"])
        return st["x"]
    if kind == "smooth":
        st["x"].copy_(st["d0"])
        s.vanka_sweep(st["top"], st["rhs"], st["x"], 2, OMEGA)
        return st["x"]
    if kind == "vcycle":
        s.vcycle(st["rhs"], st["x"], 2, 2, OMEGA)
        return st["x"]
    if kind == "newton":
        s.set_hierarchy(st["levels"], st["dim"], st["k"])
    s.build_cell_inverses(fp32=st["fp32"], full=kind == "gradient")
    s.gmres_solve(st["rhs"], st["x"], fixed_iters=st["iters"], omega=OMEGA)
    if kind != "gradient":
        return st["x"]
    s.gmres_solve_transposed(st["q"], st["lam"], fixed_iters=st["iters"], omega=OMEGA)
    # dL/dnu_c = -lam_c (W (x) K_c) x_c + lam_c F_c
    s.cell_gradient(st["top"], st["lam"], st["x"], *st["terms"], -1.0, st["cells"], st["f"], 1.0,
                    st["grad"])
    return st["x"], st["lam"], st["grad"]


# --------------------------------------------------------------------- work
def _counts(n):
    """(cells, spatial DoFs, spatial blocks) of one level's mesh."""
    d, cells = len(n), int(np.prod(n))
    dofs = d * int(np.prod([2 * c + 1 for c in n])) + (d + 1) * cells
    blocks = d * int(np.prod([8 * c + 1 for c in n])) + 2 * cells * 3 ** d * d * (d + 1)
    return cells, dofs, blocks


def _apply(n, b, factored):
    """Bytes and flops of one product with a level's operator: its values and
    columns once, three vectors."""
    _, dofs, blocks = _counts(n)
    values = 2 if factored else b * b
    return np.array([blocks * (8 * values + 4) + 24 * dofs * b,
                     2.0 * blocks * (2 * b if factored else b * b)])


def _sweep(n, b):
    """One sweep, the cell solves' operators left out: cell DoF lists and
    three vectors; one product with an inverse row per DoF."""
    cells, dofs, _ = _counts(n)
    nls = len(n) * 3 ** len(n) + len(n) + 1
    return np.array([4 * cells * nls + 24 * dofs * b, 2.0 * dofs * b * nls])


def _build(n, b):
    """Cell inverses, velocity components apart: the operator's values once,
    2 m^3 per block of m = 3^dim nodes."""
    cells, _, blocks = _counts(n)
    m = 3 ** len(n)
    return np.array([16.0 * blocks, 2.0 * m ** 3 * len(n) * b * cells])


def _cycle(meshes, b, factored):
    """V(2,2): four sweeps and four residuals per smoothed level, the first
    sweep from zero without one, and one before the restriction."""
    return sum(4 * _sweep(n, b) + 4 * _apply(n, b, factored) for n in meshes[1:]) + \
        _apply(meshes[0], b, factored)


def _hierarchy(n, levels):
    return [tuple(c >> s for c in n) for s in range(levels - 1, -1, -1)]


def work(case):
    kind, b = case["kind"], case["k"] + 1
    if kind == "batch":
        parts = [_hierarchy(n, levels) for n, levels in _batch_choice(case["n"])]
    else:
        parts = [_hierarchy(_mesh(case), case["levels"])]
    factored = kind not in ("newton", "blocks", "gradient")
    total = np.zeros(2)
    for meshes in parts:
        n = meshes[-1]
        if kind == "residual":
            total += _apply(n, b, factored)
        elif kind == "smooth":
            total += 2 * (_sweep(n, b) + _apply(n, b, factored))
        elif kind == "vcycle":
            total += _cycle(meshes, b, factored)
        else:
            total += sum(_build(m, b) for m in meshes)
            solves = 2 if kind == "gradient" else 1
            total += solves * case["iters"] * (_cycle(meshes, b, factored) + _apply(n, b, factored))
    return dict(bytes=float(total[0]), flops=float(total[1]))


# -------------------------------------------------------------------- exact
class _Exact:
    """The same operations in plain torch, 64 bits."""

    def __init__(self, geo, k, tau):
        self.b = k + 1
        self.levels = _oseen_levels(geo, k, tau)
        self.J = [self._matrix(L) for L in self.levels]
        self.inv = {}

    def _matrix(self, L):
        b = self.b
        rows = np.repeat(np.arange(L["n_sdofs"]), np.diff(L["rowptr"]))
        r, c, l = rows[:, None, None] * b, np.asarray(L["col"])[:, None, None] * b, np.arange(b)
        idx = np.stack([np.broadcast_to(r + l[None, :, None], L["val"].shape).ravel(),
                        np.broadcast_to(c + l[None, None, :], L["val"].shape).ravel()])
        n = L["n_sdofs"] * b
        return torch.sparse_coo_tensor(torch.from_numpy(idx), torch.from_numpy(L["val"].ravel()),
                                       (n, n)).coalesce().to(DEV).to_sparse_csr()

    def _cells(self, g):
        """(DoFs, inverse, owned mask) of chunks of cells: a DoF belongs to the
        last cell that holds it."""
        if g in self.inv:
            return self.inv[g]
        L, b = self.levels[g], self.b
        csd = L["cell_sdofs"]
        owner = np.zeros(L["n_sdofs"], np.int64)
        for c in range(csd.shape[0]):
            owner[csd[c]] = c
        dofs = torch.from_numpy((csd[:, :, None].astype(np.int64) * b + np.arange(b)).reshape(
            len(csd), -1)).to(DEV)
        own = torch.from_numpy(np.repeat(owner[csd] == np.arange(len(csd))[:, None], b, 1)).to(DEV)
        keys = np.repeat(np.arange(L["n_sdofs"], dtype=np.int64), np.diff(L["rowptr"])) * \
            L["n_sdofs"] + L["col"]
        keys = torch.from_numpy(keys).to(DEV)
        val = torch.from_numpy(L["val"]).to(DEV)
        out = []
        for c0 in range(0, len(csd), 512):
            sd = torch.from_numpy(csd[c0:c0 + 512].astype(np.int64)).to(DEV)
            want = sd[:, :, None] * L["n_sdofs"] + sd[:, None, :]
            pos = torch.searchsorted(keys, want.reshape(-1)).clamp_(max=len(keys) - 1)
            blk = val[pos] * (keys[pos] == want.reshape(-1))[:, None, None]
            m, nls = sd.shape
            J = blk.reshape(m, nls, nls, b, b).permute(0, 1, 3, 2, 4).reshape(m, nls * b, nls * b)
            inv = torch.linalg.inv(J.cpu()).to(DEV)
            out.append((dofs[c0:c0 + 512], inv, own[c0:c0 + 512]))
        self.inv[g] = out
        return out

    def residual(self, g, r, d):
        return r - self.J[g] @ d

    def smooth(self, g, r, d, n):
        for _ in range(n):
            rho = self.residual(g, r, d)
            new = d.clone()
            for dofs, inv, own in self._cells(g):
                c = torch.matmul(inv, rho[dofs].unsqueeze(-1)).squeeze(-1)
                new[dofs[own]] = d[dofs[own]] + OMEGA * c[own]
            d = new
        return d

    def vcycle(self, g, r):
        if g == 0:
            return torch.linalg.solve(self.J[0].to_dense(), r)
        L, b = self.levels[g], self.b
        rp, col, val = (torch.from_numpy(np.asarray(a)).to(DEV) for a in L["P"])
        P = torch.sparse_csr_tensor(rp.long(), col.long(), val,
                                    (L["n_sdofs"], self.levels[g - 1]["n_sdofs"])).to_sparse_coo()
        d = self.smooth(g, r, torch.zeros_like(r), 2)
        rc = torch.sparse.mm(P.t(), self.residual(g, r, d).reshape(-1, b)).reshape(-1)
        d = d + torch.sparse.mm(P, self.vcycle(g - 1, rc).reshape(-1, b)).reshape(-1)
        return self.smooth(g, r, d, 2)


def exact(case, seed):
    kind, k = case["kind"], case["k"]
    if kind not in ("step", "vcycle", "smooth", "residual"):
        return None
    cells, dofs, _ = _counts(_mesh(case))
    if kind == "step" and dofs * (k + 1) > 6000 or kind != "step" and cells > 28000:
        return None
    tau = _tau(k, seed)
    geo = _geometry(_mesh(case), case["levels"])
    e = _Exact(geo, k, tau)
    n, top = dofs * (k + 1), case["levels"] - 1
    if kind == "step":
        return torch.linalg.solve(e.J[top].to_dense(), _randn(n, seed))
    if kind == "vcycle":
        return e.vcycle(top, _randn(n, seed))
    rhs, d = _pair(geo, k, tau, n, seed)
    return e.smooth(top, rhs, d, 2) if kind == "smooth" else e.residual(top, rhs, d)
