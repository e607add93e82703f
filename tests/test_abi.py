"""The C-ABI library builds, loads and exports every symbol include/grg.h
declares; host-only logic (the permutation builder, parameter defaults) is
checked without a GPU."""
import ctypes as C
import os
import re
import time

import numpy as np
import pytest

import paper_0704_2341_amd as grg
from paper_0704_2341_amd import binding
from oracle import dense

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_symbols():
    with open(os.path.join(ROOT, "include", "grg.h")) as f:
        text = f.read()
    return set(re.findall(r"^\s*(?:const\s+)?\w+\s*\*?\s*(grg_\w+)\s*\(", text, re.M))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(binding.LIB_PATH):
        from paper_0704_2341_amd import build

        build.build()
    return binding.load()


def test_every_declared_symbol_is_exported(lib):
    syms = header_symbols()
    assert len(syms) >= 15
    assert syms == set(binding.EXPORTS)
    for s in syms:
        assert hasattr(lib, s), s


def test_library_is_gfx950_hip(lib):
    assert "gfx950" in grg.grg_version()


def test_params_default():
    p = grg.grg_solver_params_default()
    assert p.tol == 1e-10 and p.restart >= 1 and p.max_rhs == 12 and p.inner == grg.GRG_FP64


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (4, 6, 8, 2), (8, 8, 8, 16)])
@pytest.mark.parametrize("kind,inv", [("I", False), ("II", False), ("I", True), ("II", True)])
def test_permutation_matches_oracle(dims, kind, inv):
    q, nb = grg.grg_permutation_block(dims, 1 if kind == "I" else 2, inv)
    qo, nbo = dense.permutation_block(dims, kind, inv)
    assert nb == nbo
    assert np.array_equal(q, qo)


def test_permutation_rejects_odd_extent():
    with pytest.raises(grg.GrgError) as e:
        grg.grg_permutation_block((4, 4, 4, 5), 1)
    assert e.value.status == grg.GRG_EODD_EXTENT
    with pytest.raises(grg.GrgError) as e:
        grg.grg_permutation_block((4, 4, 4, 4), 3)
    assert e.value.status == grg.GRG_EINVAL


class _Geom(C.Structure):
    _fields_ = [("L", C.c_int * 4), ("V", C.c_int), ("Vs", C.c_int)]


class _Tune(C.Structure):
    _fields_ = [(k, C.c_int) for k in ("valid", "SB", "RG", "split", "grid", "chunk", "march")] + [("ms", C.c_float)]


def _geom(dims):
    v = int(np.prod(dims))
    return _Geom((C.c_int * 4)(*dims), v, -(-v // 256) * 256)


@pytest.mark.parametrize("dims,nrhs", [((4, 4, 4, 4), 1), ((8, 8, 8, 8), 12), ((12, 10, 9, 14), 5), ((32, 32, 32, 32), 12)])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_dc_tuning_candidates(lib, dims, nrhs, prec):
    """The defect-correction tuner times the site-parallel step at every workgroup
    size and the hop-per-wavefront form at every size of field, whatever form the
    default launch there has, and the marching forms with their own workgroups."""
    f = lib._ZN3grg13dc_candidatesERKNS_4GeomEiiPNS_10DslashTuneEi
    f.restype, f.argtypes = C.c_int, [C.POINTER(_Geom), C.c_int, C.c_int, C.POINTER(_Tune), C.c_int]
    out = (_Tune * 4096)()
    g = _geom(dims)
    n = f(C.byref(g), prec, nrhs, out, 4096)
    got = {(t.SB, t.RG, t.split, t.march, t.chunk): t.grid for t in out[:n]}
    for sb in (64, 128, 256):
        grid = min(-(-g.V // sb) * nrhs, 2048)
        assert got[sb, 1, 0, 0, 0] == max(8, -(-grid // 8) * 8), sb
    assert (64, 1, 8, 0, 0) in got
    assert all(t.SB == 64 for t in out[:n] if t.march > 0)
    assert all(t.grid >= 8 and t.grid % 8 == 0 for t in out[:n])
    assert f(C.byref(g), prec, nrhs, out, 2) == 2  # no more than there is room for


def _march_tune(lib, dims, prec, nrhs):
    f = lib._ZN3grg16canon_march_tuneERKNS_4GeomEii
    f.restype, f.argtypes = _Tune, [C.POINTER(_Geom), C.c_int, C.c_int]
    return f(C.byref(_geom(dims)), prec, nrhs)


@pytest.mark.parametrize("prec", [0, 1, 2])
def test_march_rule(lib, prec):
    """The t-march of D runs where its slices fill their tiles of 64 sites, with the
    chunks of the fewest rounds x (slices + 1), the longest among equals; the rule
    itself takes no time that grows with Lt.  The defect correction's marching
    default as well needs slices that fill their tiles."""
    rng = np.random.default_rng(75)
    for _ in range(300):
        dims = [int(d) for d in np.exp(rng.uniform(0, np.log(33), 4))]
        nrhs = int(rng.integers(1, 17))
        t = _march_tune(lib, dims, prec, nrhs)
        v3 = dims[0] * dims[1] * dims[2]
        tiles = -(-v3 // 64)
        waves = -(-v3 * dims[3] // 64) * nrhs
        assert bool(t.valid) == (waves > 512 and 4 * v3 >= 3 * 64 * tiles), (dims, nrhs)
        if t.valid:
            pairs, res = tiles * nrhs, 1024 if prec == 0 else 2048
            cost = {T: -(-pairs * -(-dims[3] // T) // res) * (T + 1) for T in range(1, dims[3] + 1)}
            best = max(T for T in cost if cost[T] == min(cost.values()))
            assert t.march == best, (dims, nrhs)
            assert t.grid == max(8, -(-min(pairs * -(-dims[3] // best), res) // 8) * 8)
    for dims in ((1, 1, 1, 1 << 27), (2, 2, 2, 8192), (3, 3, 3, 4096), (5, 13, 1, 4096)):
        assert not _march_tune(lib, dims, prec, 12).valid
        d = lib._ZN3grg15default_dc_tuneERKNS_4GeomEii
        d.restype, d.argtypes = _Tune, [C.POINTER(_Geom), C.c_int, C.c_int]
        assert d(C.byref(_geom(dims)), prec, 12).march == 0
    t0 = time.perf_counter()
    for _ in range(100):
        assert _march_tune(lib, (4, 4, 4, 1 << 21), prec, 1).valid
    assert time.perf_counter() - t0 < 0.1  # (a walk over every T: over a second)
