"""The C-ABI library builds, loads and exports every symbol include/grg.h
declares; host-only logic (the permutation builder, parameter defaults) is
checked without a GPU."""
import ctypes as C
import os
import re

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
