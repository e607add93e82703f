"""The launches that untuned handles use: on each side of the sizes at which
the default rule changes form, the stencils agree bit for bit with the plain
one-wavefront, one-hop launch (every form sums a site's hops in the same
order), and the D_rr solve agrees with the one that runs the site-parallel
defect-correction step to twice the solver tolerance times the condition
number of D_rr on these fields (about 5): 1e-9."""
import numpy as np
import pytest

from grg_inputs import gaussian_vectors

from gpu_support import Lattice, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

# 64 wavefronts; 4096 (several per SIMD); 36864 (more than the chip holds, RHS
# grouped, t-marching correction); planes of 256 columns (BF16 plane form)
SIZES = [((8, 8, 8, 8), 1), ((8, 8, 8, 32), 16), ((24, 24, 16, 16), 16), ((32, 16, 8, 8), 5)]


@pytest.mark.parametrize("dims,nrhs", SIZES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_default_launches(dims, nrhs):
    import torch

    lat = Lattice(dims, 0.5, 71)
    grg = lat.grg
    xd = to_dev(gaussian_vectors(12 * lat.V, nrhs, 71))
    yd, zd = torch.empty_like(xd), torch.empty_like(xd)
    for prec in ("fp64", "fp32", "bf16"):
        s = lat.schur(-0.2, "I", False, tol=1e-10, inner=prec, inner_tol=1e-2 if prec == "bf16" else 1e-5,
                      max_rhs=nrhs)
        print(f"default launches {dims} {prec} x {nrhs}", flush=True)
        grg.grg_block_apply(s.h, prec, 0, 0, xd, yd, nrhs)
        grg.grg_schur_set_launch(s.h, prec, nrhs, [64, 1, 1, 64, 0, 0])
        grg.grg_block_apply(s.h, prec, 0, 0, xd, zd, nrhs)
        assert torch.equal(yd, zd), prec
        for parity in (0, 1):
            s2 = lat.schur(-0.2, "I", False, inner=prec, max_rhs=nrhs)
            grg.grg_reduced_apply(s2.h, prec, parity, xd, yd, nrhs)
            grg.grg_schur_set_launch(s2.h, prec, nrhs, [64, 1, 1, 64, 0, 0], eo=True)
            grg.grg_reduced_apply(s2.h, prec, parity, xd, zd, nrhs)
            assert torch.equal(yd, zd), (prec, parity)
            s2.close()
        grg.grg_drr_solve(s.h, xd, yd, nrhs)
        grg.grg_schur_set_dc_launch(s.h, prec, nrhs, [64, 1, 0, 64, 0, 0])
        grg.grg_drr_solve(s.h, xd, zd, nrhs)
        assert rel_err(to_host(yd), to_host(zd)) < 1e-9, prec
        s.close()
    lat.close()


@pytest.mark.parametrize("dims,nrhs", [((4, 4, 4, 4), 1), ((3, 5, 2, 7), 3), ((1, 6, 1, 11), 16), ((9, 7, 10, 11), 5)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_canonical_forms(dims, nrhs):
    """The forms that read or write the canonical fields directly (the smallest
    fields, ragged tiles, extents of one) against the staged form: D in place is
    staged, and a pinned launch stages the sub-blocks; bit for bit."""
    import torch

    lat = Lattice(dims, 0.5, 72)
    grg, V = lat.grg, lat.V
    order = np.random.default_rng(72).permutation(V).astype(np.int32)
    h = grg.grg_schur_create(lat.h, -0.2, order, max(1, V // 5), grg.grg_solver_params_default(max_rhs=nrhs))
    xd = to_dev(gaussian_vectors(12 * V, nrhs, 72))
    yd, zd = torch.empty_like(xd), torch.empty_like(xd)
    for prec in ("fp64", "fp32", "bf16"):
        print(f"canonical forms {dims} {prec} x {nrhs}", flush=True)
        grg.grg_dirac_apply(lat.h, -0.2, prec, xd, yd, nrhs)
        zd.copy_(xd)
        grg.grg_dirac_apply(lat.h, -0.2, prec, zd, zd, nrhs)
        assert torch.equal(yd, zd), prec
        outs = {}
        for pinned in (False, True):
            if pinned:
                grg.grg_schur_set_launch(h, prec, nrhs, [64, 1, 0, 64, 0, 0])
            for rows in (-1, 0, 1):
                for cols in (-1, 0, 1):
                    grg.grg_block_apply(h, prec, rows, cols, xd, yd, nrhs)
                    if pinned:
                        assert torch.equal(yd, outs[rows, cols]), (prec, rows, cols)
                    else:
                        outs[rows, cols] = yd.clone()
    grg.grg_schur_destroy(h)
    lat.close()


@pytest.mark.parametrize("dims,nrhs", [((8, 8, 8, 8), 9), ((16, 4, 8, 5), 16), ((64, 2, 2, 9), 16), ((7, 31, 5, 20), 2),
                                       ((128, 3, 2, 12), 4), ((2, 3, 5, 131), 12), ((33, 32, 32, 1), 1),
                                       ((32, 32, 16, 18), 3)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_canonical_march(dims, nrhs):
    """The t-march over canonical fields: x-rows that tile the lanes and rows that do
    not, longer than a tile, ragged last tiles, time chunks with a remainder,
    one slice, one and several rounds of items; against the staged form (D in
    place), bit for bit, and outside the fields nothing is written."""
    import torch

    lat = Lattice(dims, 0.5, 73)
    grg, V = lat.grg, lat.V
    x = to_dev(gaussian_vectors(12 * V, nrhs, 73))
    room = torch.full((nrhs * 12 * V + 512,), 3.0, dtype=torch.complex128, device="cuda")
    y, z = room[256:-256].view(nrhs, 12 * V), torch.empty_like(x)
    for prec in ("fp64", "fp32", "bf16"):
        print(f"canonical march {dims} {prec} x {nrhs}", flush=True)
        for apply in (grg.grg_dirac_apply, grg.grg_dirac_apply_noalloc):
            y.fill_(7.0)
            try:
                apply(lat.h, -0.2, prec, x, y, nrhs)
            except grg.GrgError as e:
                assert apply is grg.grg_dirac_apply_noalloc and e.status == grg.GRG_ETOO_LARGE
                continue
            z.copy_(x)
            grg.grg_dirac_apply(lat.h, -0.2, prec, z, z, nrhs)
            assert torch.equal(y, z), (prec, apply)
            assert bool((room[:256] == 3.0).all()) and bool((room[-256:] == 3.0).all())
    lat.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_marching_launch_ignores_split(prec):
    """A marching launch runs as such whatever its split (8 names the hop-per-wavefront
    form only where march is 0): the sub-blocks and a solve, to the bits of split 0."""
    import torch

    dims, nrhs = (8, 8, 8, 8), 3
    lat = Lattice(dims, 0.5, 74)
    grg = lat.grg
    s = lat.schur(-0.2, "I", False, tol=1e-8, inner=prec, inner_tol=1e-2, eo=0, max_rhs=nrhs)
    x = to_dev(gaussian_vectors(12 * lat.V, nrhs, 74))
    outs = []
    for split in (0, 8):
        print(f"march 4, split {split}, {prec}", flush=True)
        grg.grg_schur_set_launch(s.h, prec, nrhs, [64, 1, split, 64, 0, 4])
        y, z = torch.empty_like(x), torch.empty_like(x)
        grg.grg_block_apply(s.h, prec, 0, -1, x, y, nrhs)
        st = grg.grg_drr_solve(s.h, x, z, nrhs)
        assert st["converged"]
        outs.append((y, z))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    for bad in ([128, 1, 8, 64, 0, 0], [64, 3, 8, 64, 0, 0], [64, 1, 8, 60, 0, 0]):
        with pytest.raises(grg.GrgError) as e:
            grg.grg_schur_set_launch(s.h, prec, nrhs, bad)
        assert e.value.status == grg.GRG_EINVAL
    s.close()
    lat.close()


@pytest.mark.parametrize("dims,nrhs", [((8, 8, 8, 9), 8), ((8, 8, 8, 8), 15), ((8, 8, 8, 18), 8), ((12, 16, 8, 16), 4)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_either_side_of_the_forms(dims, nrhs):
    """576, 960, 1152 and 1536 wavefronts, and a RHS more: 576 and 1152 are the last that
    the solves give a hop per wavefront in FP64 and FP32, 1536 (and 1024 in BF16) the
    last that the applies between canonical fields do.  Sub-blocks to the bits of the
    plain launch, and a solve whose residual meets its tolerance."""
    import torch

    lat = Lattice(dims, 0.5, 80)
    grg = lat.grg
    for n in (nrhs, nrhs + 1):
        x = to_dev(gaussian_vectors(12 * lat.V, n, 80))
        y, z = torch.empty_like(x), torch.empty_like(x)
        order = np.arange(lat.V, dtype=np.int32)
        coarse = order % 16 == 0
        q, nb = np.concatenate([order[coarse], order[~coarse]]), int(coarse.sum())
        for prec in ("fp64", "fp32", "bf16"):
            print(f"{dims} x {n} {prec}", flush=True)
            h = grg.grg_schur_create(lat.h, -0.2, q, nb, grg.grg_solver_params_default(
                tol=1e-8, inner=prec, inner_tol=1e-2, method="bicgstab", eo=0, max_rhs=n))
            st = grg.grg_drr_solve(h, x, z, n)
            assert st["converged"] and st["true_rel_resid"] <= 1e-8
            grg.grg_block_apply(h, prec, 0, -1, x, y, n)
            grg.grg_schur_set_launch(h, prec, n, [64, 1, 0, 64, 0, 0])
            grg.grg_block_apply(h, prec, 0, -1, x, z, n)
            assert torch.equal(y, z), (prec, n)
            grg.grg_schur_destroy(h)
    lat.close()
