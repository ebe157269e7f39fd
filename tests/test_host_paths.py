"""Host paths of the library that a device cannot be asked for, on a fake HIP
runtime (fake_hip.cpp) in a process of their own: memory that is not there,
exceptions of the host allocator at the C entries, grids at their limits."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
import numpy as np
sys.path.insert(0, {root!r})
fake = ctypes.CDLL({lib!r}, mode=ctypes.RTLD_GLOBAL)
fake.fake_limit.argtypes = [ctypes.c_size_t]
fake.fake_used.restype = fake.fake_peak.restype = ctypes.c_size_t
fake.fake_fail_new.argtypes = [ctypes.c_long]
fake.fake_new_left.restype = ctypes.c_long
import paper_2107_10561_amd as stv
from stgen import fe
from stgen.problem import make_problem, spatial_factors

def solver():
    s = stv.Solver.__new__(stv.Solver)
    h = ctypes.c_void_p()
    assert stv._lib.stv_create(ctypes.byref(h), 0, None) == 0
    s._h, s._torch, s.device, s.stream, s.n_st = h, None, 0, None, []
    return s

def factors(s, ps, g=0):
    _, w, C, _ = fe.time_matrices(ps[0].k)
    ma = [spatial_factors(p.levels[g]) for p in ps]
    s.set_kron_factors(g, np.concatenate([m for m, _ in ma]), np.concatenate([a for _, a in ma]),
                       np.asarray(C, dtype=np.float64), ps[0].tau * np.asarray(w, dtype=np.float64))
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", os.path.join(HERE, "fake_hip.cpp"), "-o", lib], check=True)

    def go(body):
        r = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, lib=lib) + body],
                           capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, (r.returncode, r.stdout[-2000:], r.stderr[-3000:])
        return r.stdout

    return go


@pytest.mark.parametrize("kron", [True, False])
def test_parts_that_do_not_fit(run, kron):
    """A device that holds the whole elimination's buffers but not the parts':
    the build succeeds, with the whole elimination."""
    run(f"""
p = make_problem(2, (16, 4), 1, 1, 0.01, 1e-3, 7)
s = solver()
s.set_coarse_algorithm("tournament")
s.set_hierarchy(p.levels, 2, 1)
if {kron}: factors(s, [p])
fake.fake_peak(1)
before = fake.fake_used()
s.build_cell_inverses(full=True)
whole = fake.fake_peak(0)
s.set_coarse_algorithm("auto")
s.set_hierarchy(p.levels, 2, 1)
if {kron}: factors(s, [p])
assert fake.fake_used() <= before + (1 << 20), (fake.fake_used(), before)
fake.fake_peak(1)
s.build_cell_inverses(full=True)
assert fake.fake_peak(0) > whole, "the parts take more here"
s.set_hierarchy(p.levels, 2, 1)
if {kron}: factors(s, [p])
fake.fake_limit(whole + (64 << 10))
s.build_cell_inverses(full=True)
s.build_cell_inverses(full=True)
""")


@pytest.mark.parametrize("kron", [True, False])
def test_host_allocations_that_fail(run, kron):
    """Every allocation of the host in turn fails once in set_hierarchy, in
    set_kron_factors and in the build: the call returns (with STV_ENOMEM, or
    done where a thread's job then ran in the caller), leaves no device memory
    behind, and the same call succeeds afterwards."""
    out = run(f"""
p = make_problem(2, (32, 8), 2, 1, 0.01, 1e-3, 7)
arr, keep = stv._marshal_levels(p.levels)
s = solver()
lib = stv._lib
_, w, C, _ = fe.time_matrices(1)
C = np.ascontiguousarray(C, dtype=np.float64)
tw = np.ascontiguousarray(p.tau * np.asarray(w, dtype=np.float64))
ma = [tuple(np.ascontiguousarray(v, dtype=np.float64) for v in spatial_factors(L)) for L in p.levels]
hier = lambda: lib.stv_set_hierarchy(s._h, 2, 2, 1, arr)
fact = lambda: lib.stv_set_kron_factors(s._h, 0, ma[0][0].ctypes.data, ma[0][1].ctypes.data,
                                        C.ctypes.data, tw.ctypes.data)
build = lambda: lib.stv_build_cell_inverses(s._h, 0, None, None)
calls = [("hier", lambda: None, hier), ("build", hier, build)]
if {kron}:
    calls = [("fact", hier, fact), ("build", lambda: (hier(), fact()), build)]
for name, before, call in calls:
    n, failed = 0, 0
    while True:
        if name != "hier":
            before()
        base = fake.fake_used()
        fake.fake_fail_new(n)
        rc = call()
        left = fake.fake_new_left()
        fake.fake_fail_new(-1)
        if left >= 0:           # fewer allocations than that: the last one
            assert rc == 0, (name, n, rc)
            break
        assert rc in (0, stv.STV_ENOMEM), (name, n, rc)
        failed += rc != 0
        if rc != 0:
            if name == "hier":
                assert fake.fake_used() <= (1 << 20), (name, n, fake.fake_used())
            else:
                assert fake.fake_used() <= base + (1 << 16), (name, n, fake.fake_used(), base)
            if n % 16 == 0:
                if name == "build":
                    before()
                assert call() == 0, (name, n)
        n += 1 if n < 200 else 7
    print(name, n, failed)
    assert failed > 5
""")
    print(out)


@pytest.mark.parametrize("cap,grid", [(0, 256), (7, 7), (-1, 160), (1000, 256)])
def test_cap_of_the_cell_inverses(run, cap, grid):
    """STV_OPT_INVERSE_CUS holds for 3d cells eliminated by component: at most
    that many workgroups of four cells (-1: five eighths of 256)."""
    run(f"""
p = make_problem(3, (16, 8, 8), 2, 1, 0.01, 1e-3, 7)
s = solver()
s.set_hierarchy(p.levels, 3, 1)
for g in (0, 1): factors(s, [p], g)
s.set_inverse_cus({cap})
s.build_cell_inverses()
assert fake.fake_grid(b"k_inverse_comp") == {grid}, fake.fake_grid(b"k_inverse_comp")
""")


@pytest.mark.parametrize("cells,levels,last", [((16, 8, 8), 4, 0), ((16, 4, 4), 2, 224)])
def test_cells_in_launches_beside_the_chain_only(run, cells, levels, last):
    """3d cells without factors: launches of at most 224 cells while the coarse
    chain is expected to last (8x2x2 coarse cells: all 256), the others at once
    (2x1x1 coarse cells, 1,024 finest ones)."""
    run(f"""
p = make_problem(3, {cells}, {levels}, 1, 0.01, 1e-3, 7)
s = solver()
s.set_hierarchy(p.levels, 3, 1)
s.build_cell_inverses()
g = fake.fake_grid(b"k_inverse_mfma")
assert {last} == 0 and g > 224 or 0 < g <= {last}, g
""")
