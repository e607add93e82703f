"""The second-order Schur complement approximation of section 3 on the GPU
against the oracle: dense at 4^4 for all four permutations, matrix-free at
larger volumes with several right-hand sides, and the clustering of the
spectrum of S~_bb^{-1} S_bb around one that section 4 uses it for; and the
approximation that ignores the couplings inside D_rr, dense and matrix-free,
with its free-field spectrum in closed form."""
import numpy as np
import pytest

from grg_inputs import gaussian_vectors, su3_links
from oracle import dense, matfree

from gpu_support import Lattice, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

PERMS = [("I", False), ("II", False), ("I", True), ("II", True)]


@pytest.fixture(scope="module")
def small():
    lat = Lattice((4, 4, 4, 4), 0.4, 1)
    yield lat, dense.wilson_dense(lat.links, lat.dims, 0.1)
    lat.close()


@pytest.mark.parametrize("kind,inv", PERMS)
def test_dense_4x4x4x4(small, kind, inv):
    lat, d = small
    s = lat.schur(0.1, kind, inv, tol=1e-13, max_rhs=12)
    got = lat.grg.grg_reusken_assemble(s.h, s.nb)
    want = dense.reusken_dense(d, s.q, s.nb)
    assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()
    # section 4: the spectrum of S~^{-1} S clusters around one
    ex = lat.grg.grg_schur_assemble(s.h, s.nb)
    ev = np.linalg.eigvals(np.linalg.solve(got, ex))
    assert np.abs(ev - 1).max() < 0.25, np.abs(ev - 1).max()
    s.close()


@pytest.mark.parametrize("dims,kind,inv,nrhs", [((8, 8, 8, 8), "II", True, 4),
                                                ((8, 6, 4, 10), "I", False, 3),
                                                ((16, 16, 16, 16), "I", True, 12)])
def test_matrix_free(dims, kind, inv, nrhs):
    import torch

    lat = Lattice(dims, 0.5, 2)
    s = lat.schur(-0.2, kind, inv, max_rhs=nrhs)
    xb = gaussian_vectors(12 * s.nb, nrhs, 2)
    x = to_dev(xb)
    y = torch.empty_like(x)
    lat.grg.grg_reusken_apply(s.h, x, y, nrhs)
    got = to_host(y)
    sample = [0, nrhs - 1]
    want = matfree.reusken_apply(lat.links, dims, -0.2, s.q, s.nb, xb[sample])
    assert rel_err(got[sample], want) < 1e-12
    s.close()
    lat.close()


def test_new_gauge_field_recomputes_row_sums():
    """The row sums d~ = D_rr 1 are kept between applies: a new gauge field
    on the lattice must replace them (the apply after it matches the oracle
    on the new links, not the old)."""
    import torch

    from grg_inputs import su3_links

    dims, nrhs = (8, 8, 4, 8), 2
    lat = Lattice(dims, 0.5, 5)
    s = lat.schur(-0.2, "II", True, max_rhs=nrhs)
    xb = gaussian_vectors(12 * s.nb, nrhs, 6)
    x = to_dev(xb)
    y = torch.empty_like(x)
    lat.grg.grg_reusken_apply(s.h, x, y, nrhs)
    first = to_host(y)
    links2 = su3_links(dims, 0.5, 7)
    lat.grg.grg_gauge_set(lat.h, links2)
    lat.grg.grg_reusken_apply(s.h, x, y, nrhs)
    got = to_host(y)
    want = matfree.reusken_apply(links2, dims, -0.2, s.q, s.nb, xb)
    assert rel_err(got, want) < 1e-12
    assert rel_err(first, want) > 1e-3  # the field did change the operator
    s.close()
    lat.close()


def test_zero_diagonal_rejected():
    import torch

    lat = Lattice((4, 4, 4, 4), 0.4, 1)
    s = lat.schur(-4.0, "I", False, max_rhs=1)
    x = torch.zeros(12 * s.nb, dtype=torch.complex128, device="cuda")
    with pytest.raises(lat.grg.GrgError):
        lat.grg.grg_reusken_apply(s.h, x, torch.empty_like(x), 1)
    with pytest.raises(lat.grg.GrgError):
        lat.grg.grg_diag_schur_apply(s.h, x, torch.empty_like(x), 1)
    s.close()
    lat.close()


# ------------------------------------------------------------------ ignoring D_rr
@pytest.mark.parametrize("kind,inv", PERMS)
def test_diag_schur_dense_4x4x4x4(small, kind, inv):
    """D_bb - D_br D_rb / d assembled on the GPU against the dense oracle.
    On the all-even coarse set (Type I, and forward Type II, which has the
    same set) the second-order correction vanishes identically: D_rb lands on
    sites with one odd coordinate, a hop inside D_rr on sites with two, and no
    coarse site is one hop from those, so S~_bb = S0_bb there."""
    lat, d = small
    s = lat.schur(0.1, kind, inv, tol=1e-13, max_rhs=12)
    got = lat.grg.grg_diag_schur_assemble(s.h, s.nb)
    want = dense.diag_schur_dense(d, s.q, s.nb)
    assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()
    if not inv:
        second = lat.grg.grg_reusken_assemble(s.h, s.nb)
        assert np.abs(second - got).max() <= 1e-12 * np.abs(got).max()
    s.close()


def test_diag_schur_free_field_spectrum():
    """Free field, Type I: the spectrum of the GPU-assembled operator against
    its closed form d - (sum cos k)/d +- i sqrt(sum sin^2 k)/d."""
    from test_oracle_pins import same_multiset
    from test_oracle_reusken import free_diag_schur_type1_spectrum

    dims = (4, 4, 4, 4)
    links = np.zeros((256, 4, 3, 3), dtype=np.complex128)
    links[:] = np.eye(3)
    lat = Lattice(dims, 0.0, 0, links=links)
    s = lat.schur(0.1, "I", False, max_rhs=12)
    got = lat.grg.grg_diag_schur_assemble(s.h, s.nb)
    ok, worst = same_multiset(np.linalg.eigvals(got), free_diag_schur_type1_spectrum(dims, 0.1), 1e-10)
    assert ok, worst
    s.close()
    lat.close()


@pytest.mark.parametrize("dims,kind,inv,nrhs", [((8, 8, 8, 8), "II", True, 4),
                                                ((8, 6, 4, 10), "I", False, 3),
                                                ((16, 16, 16, 16), "II", False, 12)])
def test_diag_schur_matrix_free(dims, kind, inv, nrhs):
    import torch

    lat = Lattice(dims, 0.5, 3)
    s = lat.schur(-0.2, kind, inv, max_rhs=nrhs)
    xb = gaussian_vectors(12 * s.nb, nrhs, 3)
    x = to_dev(xb)
    y = torch.empty_like(x)
    lat.grg.grg_diag_schur_apply(s.h, x, y, nrhs)
    got = to_host(y)
    sample = [0, nrhs - 1]
    want = matfree.diag_schur_apply(lat.links, dims, -0.2, s.q, s.nb, xb[sample])
    assert rel_err(got[sample], want) < 1e-12
    s.close()
    lat.close()


@pytest.mark.parametrize("dims,kind,nrhs", [((4, 4, 4, 4), "first", 1), ((5, 3, 7, 4), "third", 2),
                                            ((5, 3, 7, 4), "all but one", 3), ((6, 6, 6, 6), "one", 16)])
def test_boundary_forms(dims, kind, nrhs):
    """Coarse sets whose boundary (the rest sites next to a coarse site) is a
    few sites, most of the lattice or one site, on odd extents too, in place
    and not; both approximations."""
    import torch

    lat = Lattice(dims, 0.5, 3)
    grg, V = lat.grg, lat.V
    order = np.random.default_rng(3).permutation(V).astype(np.int32)
    nb = {"first": 64, "third": V // 3, "all but one": V - 1, "one": 1}[kind]
    h = grg.grg_schur_create(lat.h, -0.2, order, nb, grg.grg_solver_params_default(max_rhs=nrhs))
    xb = gaussian_vectors(12 * nb, nrhs, 3)
    want = matfree.reusken_apply(lat.links, dims, -0.2, order, nb, xb)
    x = to_dev(xb)
    y = torch.empty_like(x)
    print(f"boundary forms {dims} {kind}", flush=True)
    grg.grg_reusken_apply(h, x, y, nrhs)
    assert rel_err(to_host(y), want) < 1e-12
    grg.grg_diag_schur_apply(h, x, y, nrhs)
    z = x.clone()
    grg.grg_diag_schur_apply(h, z, z, nrhs)
    assert torch.equal(z, y)
    z = x.clone()
    grg.grg_reusken_apply(h, z, z, nrhs)
    assert rel_err(to_host(z), want) < 1e-12
    grg.grg_schur_destroy(h)
    lat.close()


def test_zero_row_sums():
    """A free field at m0 = 0, periodic: the row sums of D_rr vanish on the
    rest sites that are not next to a coarse site, where the formula divides
    zero by zero, and its neighbours' output is not a number."""
    import torch

    dims = (8, 8, 4, 4)
    V = int(np.prod(dims))
    links = np.tile(np.eye(3, dtype=complex), (V, 4, 1, 1))
    lat = Lattice(dims, 0, 0, bc=(1, 1, 1, 1), links=links)
    s = lat.schur(0.0, "I", False, max_rhs=2)
    x = to_dev(gaussian_vectors(12 * s.nb, 2, 5))
    y = torch.empty_like(x)
    lat.grg.grg_reusken_apply(s.h, x, y, 2)
    assert bool(torch.isnan(torch.view_as_real(y)).all())
    lat.grg.grg_diag_schur_apply(s.h, x, y, 2)
    assert bool(torch.isfinite(torch.view_as_real(y)).all())
    s.close()
    lat.close()


@pytest.mark.parametrize("linked", [False, True])
def test_formula_order(linked):
    """(y - z) / d + t where the row sums equal d, so that z is y up to rounding:
    links 1 along x in the rows of coarse sites and 0 elsewhere, and a source of whole
    numbers on the sites x = 0, whose image on x = 2 and 6 is -1/2 (1 -/+ g_x) x / d.
    In units of u = 2^-53: t = y d / d^2 errs by at most 3 u, z = d t by 4, y - z is
    exact and takes t's error out again, which leaves z's rounding and the last sum's,
    and the hop to the coarse site adds two equal terms, exactly: 2 u and the second
    order.  (y / d + t first and z / d off afterwards reaches 2.9 u.)  With `linked`, a
    coarse site more whose neighbours lie next to the boundary's (z formed in a pass
    of its own)."""
    import torch

    dims, m0, nrhs = (8, 4, 4, 4), -0.45, 5
    V, d = int(np.prod(dims)), 4.0 + m0
    c = np.array([[(s // int(np.prod(dims[:mu]))) % dims[mu] for mu in range(4)] for s in range(V)])
    row = (c[:, 1:] % 2 == 0).all(axis=1)
    links = np.zeros((V, 4, 3, 3), complex)
    links[row, 0] = np.eye(3)
    coarse = row & (c[:, 0] % 2 == 0)
    if linked:
        coarse |= (c == (1, 1, 1, 0)).all(axis=1)
    q = np.concatenate([np.flatnonzero(coarse), np.flatnonzero(~coarse)]).astype(np.int32)
    nb = int(coarse.sum())
    lat = Lattice(dims, 0.0, 0, bc=(1, 1, 1, 1), links=links)
    h = lat.grg.grg_schur_create(lat.h, m0, q, nb, lat.grg.grg_solver_params_default(max_rhs=nrhs))
    cc = c[q[:nb]]
    src = np.flatnonzero(row[q[:nb]] & (cc[:, 0] == 0))
    rng = np.random.default_rng(76)
    up = rng.integers(1, 1 << 20, (nrhs, len(src), 2, 3, 2)).astype(float)  # spins 0 and 1
    xb = np.zeros((nrhs, nb, 4, 3), complex)
    xb[:, src, :2] = up[..., 0] + 1j * up[..., 1]
    x = to_dev(xb.reshape(nrhs, -1))
    y = torch.empty_like(x)
    lat.grg.grg_reusken_apply(h, x, y, nrhs)
    got = to_host(y).reshape(nrhs, nb, 4, 3)
    u0, u1 = xb[:, src, 0], xb[:, src, 1]
    checked = 0
    for xs, sg in ((2, 1), (6, -1)):
        # from x = 0 on to x + 2: -1/2 (1 + g_x) x; back to x - 2: -1/2 (1 - g_x) x
        at = np.flatnonzero(row[q[:nb]] & (cc[:, 0] == xs))
        assert (cc[at, 1:] == cc[src, 1:]).all()
        num = np.stack([u0, u1, sg * -1j * u1, sg * -1j * u0], axis=2)
        for part in (np.real, np.imag):
            want = part(num).astype(np.longdouble) * np.longdouble(-0.5) / np.longdouble(d)
            err = np.abs(part(got[:, at]).astype(np.longdouble) - want) / np.abs(want)
            assert float(err.max()) <= 2.0 * 2.0 ** -53 * (1 + 1e-3), float(err.max()) * 2.0 ** 53
            checked += err.size
    assert checked == nrhs * len(src) * 2 * 24
    lat.grg.grg_schur_destroy(h)
    lat.close()


@pytest.mark.parametrize("dims,kind,inv", [((8, 8, 8, 8), "I", False), ((8, 6, 4, 10), "II", True),
                                           ((16, 16, 16, 16), "I", False), ((2, 4, 2, 2), "I", True)])
def test_first_calls(dims, kind, inv):
    """A handle's first call and the first on a new gauge field (whose row sums may
    couple sites that the last one's did not) do not know yet how many boundary sites
    there are, nor whether any are linked: to the bits of a call that does."""
    import torch

    lat = Lattice(dims, 0.5, 77)
    grg, nrhs = lat.grg, 3
    q, nb = grg.grg_permutation_block(dims, 1 if kind == "I" else 2, inv)
    x = to_dev(gaussian_vectors(12 * nb, nrhs, 77))
    links2 = su3_links(dims, 0.5, 78)
    applies = (grg.grg_reusken_apply, grg.grg_diag_schur_apply)

    def twice(h, apply):
        ys = []
        for _ in range(2):
            y = torch.empty_like(x)
            apply(h, x, y, nrhs)
            ys.append(y)
        assert torch.equal(ys[0], ys[1])
        return ys[0]

    seen = {}
    for order in (applies, applies[::-1]):
        grg.grg_gauge_set(lat.h, lat.links)
        h = grg.grg_schur_create(lat.h, -0.2, q, nb, grg.grg_solver_params_default(max_rhs=nrhs))
        for field in (0, 1):
            if field:
                grg.grg_gauge_set(lat.h, links2)
            for apply in order:
                print(f"first call {dims} {kind} {inv} {apply.__name__} field {field}", flush=True)
                y = twice(h, apply)
                assert torch.equal(seen.setdefault((apply, field), y), y)
        grg.grg_schur_destroy(h)
    sample = to_host(x)
    for field, links in ((0, lat.links), (1, links2)):
        want = matfree.reusken_apply(links, dims, -0.2, q, nb, sample)
        assert rel_err(to_host(seen[applies[0], field]), want) < 1e-12
    lat.close()


def test_first_calls_allocate_no_tables():
    """The boundary's tables lie in the handle's own memory: the first call without
    row sums allocates nothing on the device, the first one with them that field alone."""
    import torch

    dims = (24, 24, 24, 24)
    lat = Lattice(dims, 0.5, 79)
    grg = lat.grg
    q, nb = grg.grg_permutation_block(dims, 1, False)
    h = grg.grg_schur_create(lat.h, -0.2, q, nb, grg.grg_solver_params_default(max_rhs=1))
    x = to_dev(gaussian_vectors(12 * nb, 1, 79))
    y = torch.empty_like(x)
    torch.cuda.synchronize()
    free = [torch.cuda.mem_get_info()[0]]
    for apply in (grg.grg_diag_schur_apply, grg.grg_reusken_apply):
        apply(h, x, y, 1)
        free.append(torch.cuda.mem_get_info()[0])
    assert free[1] == free[0]
    rows = lat.V * 12 * 16
    assert rows <= free[1] - free[2] < rows + (1 << 21)  # (2 MiB: the allocator's unit)
    grg.grg_schur_destroy(h)
    lat.close()
