"""The workloads this library's speed is judged by, and how each is run.

A case is a dict of plain values.  `listed()` names the fixed ones, `draw()`
gives more of the same ranges, `prepare()` builds what a program holds before
the call (gauge field, handles, inputs), `run()` is one call of the public
entry points, `work()` the bytes and operations that call cannot do without,
and `exact()` the same result in 64 bits from plain torch, without the library.

Kinds:
  dirac    grg_dirac_apply: y = D x on a whole lattice
  schur    grg_schur_apply: y_b = S_bb x_b, the coarse operator (a D_rr solve inside)
  drr      grg_drr_solve: z = D_rr^-1 b
  approx   grg_reusken_apply: the second-order approximation of S_bb, no solve
  learned  grg_schur_apply with a network as the inner solve's preconditioner
  grad     grg_precond_loss_grad: the network forward and backward
  vcycle   grg_vcycle_solve: D x = f, preconditioned by the V-cycle
  batch    grg_batch_apply: S_bb of many lattices at once
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_0704_2341_amd as grg

DEV = "cuda"
EPS = 0.5                      # roughness of the synthetic links
BC = (1, 1, 1, -1)             # antiperiodic in t, as everywhere in this repository
TOL = 1e-10                    # the solver tolerance of the benchmark
INNER_TOL = {"bf16": 1e-2, "fp32": 1e-5, "fp64": 1e-5}
BATCH_SHAPES = ((8, 8, 8, 8), (12, 12, 12, 12), (16, 16, 16, 16), (8, 8, 8, 16))
CHANNELS = (4, 8, 8, 4)


def _case(name, kind, dims, nrhs, **kw):
    c = {"kind": kind, "lx": dims[0], "ly": dims[1], "lz": dims[2], "lt": dims[3], "nrhs": nrhs}
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one field on the 4^4 lattice of the dense comparisons
        _case("dirac_4x4x4x4_fp64_1", "dirac", (4, 4, 4, 4), 1, prec="fp64", m0=0.1),
        # odd extents and an odd number of fields: no even-odd form, ragged tiles
        _case("dirac_15x9x11x22_fp32_5", "dirac", (15, 9, 11, 22), 5, prec="fp32", m0=-0.2),
        # the benchmark's lattice: a propagator's twelve fields through D
        _case("dirac_32x32x32x32_fp64_12", "dirac", (32, 32, 32, 32), 12, prec="fp64", m0=-0.3),
        # a small coarse-operator call: one source, launches and waits count
        _case("schur_8x8x8x8_bf16_1", "schur", (8, 8, 8, 8), 1, prec="bf16", m0=-0.2, perm=1, inv=False,
              tune=False),
        # the 16^4 workload with eight right-hand sides on an inverse ordering, FP32 inner solve
        _case("schur_16x16x16x16_fp32_8", "schur", (16, 16, 16, 16), 8, prec="fp32", m0=-0.2, perm=2, inv=True,
              tune=False),
        # the benchmark: S_bb at 32^4, twelve right-hand sides, BF16 inner solve, tuned
        _case("schur_32x32x32x32_bf16_12", "schur", (32, 32, 32, 32), 12, prec="bf16", m0=-0.3, perm=1, inv=False,
              tune=True),
        # the paper's solver on a lattice with odd extents (no even-odd reduction)
        _case("drr_12x10x9x14_bicgstab_fp64_4", "drr", (12, 10, 9, 14), 4, prec="fp64", m0=-0.2),
        # the approximation of section 3 at the benchmark's size
        _case("approx_32x32x32x32_12", "approx", (32, 32, 32, 32), 12, m0=-0.3, perm=1, inv=False),
        # the learned preconditioner inside the solve
        _case("learned_16x16x16x16_12", "learned", (16, 16, 16, 16), 12, prec="bf16", m0=-0.3, perm=1, inv=False),
        # one training step's loss and gradients: the network forward and backward
        _case("grad_16x16x16x16_12", "grad", (16, 16, 16, 16), 12, m0=-0.3, perm=1, inv=False),
        # section 4's experiment: many short kernels on a small lattice
        _case("vcycle_8x8x8x8_4", "vcycle", (8, 8, 8, 8), 4, m0=-1.0, levels=3, perm=1, inv=False),
        # 48 lattices of mixed sizes, four right-hand sides each, in one graph
        _case("batch_48_fp32_4", "batch", (0, 0, 0, 0), 4, prec="fp32", count=48),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _even(rng, lo, hi):
    return 2 * _log_int(rng, lo // 2, hi // 2)


def draw(rng):
    kind = rng.choice(("dirac", "dirac", "schur", "schur", "schur", "drr", "approx", "learned", "grad", "vcycle",
                       "batch"))
    m0 = round(rng.uniform(-0.3, 0.1), 3)
    perm, inv = rng.choice((1, 2)), rng.choice((False, True))
    if kind == "dirac":
        dims = [_log_int(rng, 3, 32) for _ in range(4)]
        return _case(None, kind, dims, _log_int(rng, 1, 16), prec=rng.choice(("fp64", "fp32", "bf16")), m0=m0)
    if kind == "schur":
        prec = rng.choice(("bf16", "bf16", "fp32", "fp64"))
        dims = [_even(rng, 4, {"bf16": 24, "fp32": 20, "fp64": 16}[prec]) for _ in range(4)]
        return _case(None, kind, dims, _log_int(rng, 1, 12), prec=prec, m0=m0, perm=perm, inv=inv, tune=False)
    if kind == "drr":
        dims = [_log_int(rng, 3, 20) for _ in range(4)]
        return _case(None, kind, dims, _log_int(rng, 1, 12), prec=rng.choice(("fp64", "fp32")), m0=m0)
    if kind == "approx":
        dims = [_even(rng, 4, 28) for _ in range(4)]
        return _case(None, kind, dims, _log_int(rng, 1, 12), m0=m0, perm=perm, inv=inv)
    if kind in ("learned", "grad"):
        dims = [_even(rng, 4, 18) for _ in range(4)]
        c = _case(None, kind, dims, _log_int(rng, 2, 12), m0=m0, perm=perm, inv=inv)
        if kind == "learned":
            c["prec"] = "bf16"
        return c
    if kind == "vcycle":
        dims = [8, 8, 8, 8]
        dims[rng.randrange(4)] = rng.choice((8, 16, 24))
        return _case(None, kind, dims, _log_int(rng, 1, 4), m0=round(rng.uniform(-1.0, -0.5), 3),
                     levels=rng.choice((2, 3)), perm=1, inv=False)
    return _case(None, kind, (0, 0, 0, 0), _log_int(rng, 1, 6), prec=rng.choice(("fp32", "bf16")),
                 count=_log_int(rng, 4, 32))


# ------------------------------------------------------------------ inputs
def _dims(case):
    return (case["lx"], case["ly"], case["lz"], case["lt"])


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _gauss(shape, gen):
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=gen, device=DEV, dtype=torch.float64))


def _mm3(a, b):
    """Products of 3x3 matrices, as element-wise sums."""
    return sum(a[..., :, k, None] * b[..., None, k, :] for k in range(3))


def _links(volume, gen):
    """SU(3) links, (V, 4, 3, 3): exp(i EPS sum_k a_k lambda_k), a_k ~ N(0, 1), made unitary again by
    Gram-Schmidt, as the repository's generator makes them."""
    a = EPS * torch.randn((volume * 4, 8), generator=gen, device=DEV, dtype=torch.float64)
    h = torch.zeros((volume * 4, 3, 3), device=DEV, dtype=torch.complex128)
    s3 = 1 / math.sqrt(3.0)
    h[:, 0, 0] = a[:, 2] + s3 * a[:, 7]
    h[:, 1, 1] = -a[:, 2] + s3 * a[:, 7]
    h[:, 2, 2] = -2 * s3 * a[:, 7]
    for (i, j), (k, l) in (((0, 1), (0, 1)), ((0, 2), (3, 4)), ((1, 2), (5, 6))):
        h[:, i, j] = torch.complex(a[:, k], -a[:, l])
        h[:, j, i] = torch.complex(a[:, k], a[:, l])
    h = h * (1j / 16)
    one = torch.eye(3, device=DEV, dtype=torch.complex128).expand_as(h)
    u = one
    for k in range(10, 0, -1):     # the series of exp(i H / 16), then four squarings
        u = one + _mm3(h, u) / k
    for _ in range(4):
        u = _mm3(u, u)
    r0 = u[:, 0] / u[:, 0].abs().square().sum(-1, keepdim=True).sqrt()
    r1 = u[:, 1] - (r0.conj() * u[:, 1]).sum(-1, keepdim=True) * r0
    r1 = r1 / r1.abs().square().sum(-1, keepdim=True).sqrt()
    r2 = torch.stack([r0[:, 1] * r1[:, 2] - r0[:, 2] * r1[:, 1], r0[:, 2] * r1[:, 0] - r0[:, 0] * r1[:, 2],
                      r0[:, 0] * r1[:, 1] - r0[:, 1] * r1[:, 0]], -1).conj()
    return torch.stack([r0, r1, r2], -2).reshape(volume, 4, 3, 3).contiguous()


def _ordering(case, dims):
    """(q, n_coarse).  Extents that the block permutations refuse get a coarse set of every sixteenth site."""
    if all(d % 2 == 0 for d in dims):
        return grg.grg_permutation_block(dims, case.get("perm", 1), case.get("inv", False))
    s = np.arange(int(np.prod(dims)), dtype=np.int32)
    coarse = s % 16 == 0
    return np.concatenate([s[coarse], s[~coarse]]), int(coarse.sum())


def _coarse_mask(q, nb, volume):
    m = np.zeros(volume, bool)
    m[q[:nb]] = True
    return torch.from_numpy(m).to(DEV)


def _batch_members(case, seed):
    """(extents, m0) per lattice: the shapes in equal shares, in an order that the seed gives, so that every
    seed's batch has the same work."""
    rng = np.random.default_rng(int(seed))
    shape = rng.permutation(np.arange(case["count"]) % len(BATCH_SHAPES))
    m0 = rng.uniform(-0.3, 0.1, size=case["count"])
    return [(BATCH_SHAPES[int(p)], float(m)) for p, m in zip(shape, m0)]


def _inputs(case, seed):
    """Everything that the seed determines: links, orderings, right-hand sides."""
    gen = _gen(seed)
    kind, n = case["kind"], case["nrhs"]
    if kind == "batch":
        members = []
        for dims, m0 in _batch_members(case, seed):
            v = int(np.prod(dims))
            q, nb = grg.grg_permutation_block(dims, 1, False)
            members.append({"dims": dims, "m0": m0, "links": _links(v, gen), "q": q, "n_coarse": nb})
        x = [_gauss((n, 12 * m["n_coarse"]), gen) for m in members]
        return {"members": members, "x": x}
    dims = _dims(case)
    v = int(np.prod(dims))
    d = {"dims": dims, "V": v, "links": _links(v, gen)}
    if kind in ("dirac", "vcycle"):
        d["x"] = _gauss((n, 12 * v), gen)
        return d
    d["q"], d["nb"] = _ordering(case, dims)
    if kind in ("drr", "grad"):
        rest = (~_coarse_mask(d["q"], d["nb"], v)).repeat_interleave(12)
        d["x"] = _gauss((n, 12 * v), gen) * rest
        if kind == "grad":
            # residual and error of comparable size, partly aligned, as a solver's pairs are
            d["e"] = (0.25 * d["x"] + 0.1 * _gauss((n, 12 * v), gen)) * rest
    else:
        d["x"] = _gauss((n, 12 * d["nb"]), gen)
    return d


def _gammas():
    g = np.zeros((4, 4, 4), complex)   # x, y, z, t in the DeGrand-Rossi basis
    b = ([[0, 1j], [1j, 0]], [[0, -1], [1, 0]], [[1j, 0], [0, -1j]], [[1, 0], [0, 1]])
    for mu in range(4):
        g[mu, :2, 2:] = b[mu]
        g[mu, 2:, :2] = np.conj(np.array(b[mu])).T
    return g


def _weights(case):
    """A network that approximates 1 / D: 1 + k + k^2 + k^3 = (1 + k)(1 + i k)(1 - i k) with k the hops over
    4 + m0, one factor per layer."""
    g = _gammas()
    d = 4.0 + case["m0"]
    flat = []
    for (fi, fo), c in zip(zip(CHANNELS[:-1], CHANNELS[1:]), (1.0, 1j, -1j)):
        w = np.zeros((9, fo, fi), complex)
        w[0, :4, :4] = np.eye(4)
        for mu in range(4):
            w[1 + 2 * mu, :4, :4] = c * 0.5 * (np.eye(4) - g[mu]) / d
            w[2 + 2 * mu, :4, :4] = c * 0.5 * (np.eye(4) + g[mu]) / d
        flat.append(w)
    flat[-1] = flat[-1] / d
    return flat


class _Held:
    """Library handles, given back with the state that holds them."""

    def __init__(self):
        self._undo = []

    def add(self, handle, destroy):
        self._undo.append((destroy, handle))
        return handle

    def __del__(self):
        while self._undo:
            destroy, handle = self._undo.pop()
            destroy(handle)


def prepare(case, seed):
    kind, n = case["kind"], case["nrhs"]
    d = _inputs(case, seed)
    held = _Held()
    s = {"case": case, "held": held}
    if kind == "batch":
        members = [dict(m, links=m["links"].cpu().numpy()) for m in d["members"]]
        prm = grg.grg_solver_params_default(tol=TOL, inner=case["prec"], inner_tol=INNER_TOL[case["prec"]],
                                            check_every=4)
        s["h"] = held.add(grg.grg_batch_create(members, n, prm), grg.grg_batch_destroy)
        s["x"] = torch.cat([x.reshape(-1) for x in d["x"]])
        s["y"] = torch.empty_like(s["x"])
        return s
    s["x"], s["y"] = d["x"], torch.empty_like(d["x"])
    lat = s["lat"] = held.add(grg.grg_lattice_create(d["dims"], BC), grg.grg_lattice_destroy)
    grg.grg_gauge_set(lat, d["links"])
    if kind == "dirac":
        return s
    if kind == "vcycle":
        prm = grg.grg_vcycle_params_default(levels=case["levels"], max_rhs=n)
        s["h"] = held.add(grg.grg_vcycle_create(lat, case["m0"], prm), grg.grg_vcycle_destroy)
        return s
    kw = {"tol": TOL, "max_rhs": n, "max_iter": 4000}
    if kind in ("schur", "learned", "drr"):
        kw.update(inner=case["prec"], inner_tol=INNER_TOL[case["prec"]])
    if kind in ("schur", "learned"):
        kw.update(check_every=2)
    if kind == "drr":
        kw.update(method="bicgstab")
    if kind == "grad":
        kw.update(inner="bf16", inner_tol=1e-2)
    h = s["h"] = held.add(grg.grg_schur_create(lat, case["m0"], d["q"], d["nb"], grg.grg_solver_params_default(**kw)),
                          grg.grg_schur_destroy)
    if case.get("tune"):
        grg.grg_schur_tune(h, n)
    if kind in ("learned", "grad"):
        p = s["net"] = held.add(grg.grg_precond_create(h), grg.grg_precond_destroy)
        grg.grg_precond_set_weights(p, np.concatenate([w.reshape(-1) for w in _weights(case)]))
        if kind == "learned":
            grg.grg_schur_attach_precond(h, p)
        else:
            s["e"] = d["e"]
    return s


def run(s):
    case = s["case"]
    kind, n = case["kind"], case["nrhs"]
    x, y = s["x"], s.get("y")
    if kind == "dirac":
        grg.grg_dirac_apply(s["lat"], case["m0"], case["prec"], x, y, n)
    elif kind in ("schur", "learned"):
        grg.grg_schur_apply(s["h"], x, y, n)
    elif kind == "drr":
        grg.grg_drr_solve(s["h"], x, y, n)
    elif kind == "approx":
        grg.grg_reusken_apply(s["h"], x, y, n)
    elif kind == "grad":
        loss, grad = grg.grg_precond_loss_grad(s["net"], x, s["e"], n)
        return {"loss": float(loss), "grad": grad}
    elif kind == "vcycle":
        grg.grg_vcycle_solve(s["h"], x, y, n, tol=1e-8)
    else:
        grg.grg_batch_apply(s["h"], x, y)
    return y


# ------------------------------------------------------------------ bytes and operations
HOP_FLOPS = 1320               # the stencil's operations per site and field


def work(case):
    kind, n = case["kind"], case["nrhs"]
    if kind == "batch":
        shapes = [BATCH_SHAPES[i % len(BATCH_SHAPES)] for i in range(case["count"])]
        v = sum(int(np.prod(d)) for d in shapes)
    else:
        v = int(np.prod(_dims(case)))
    field, coarse, links = v * 192, v // 16 * 192, v * 576
    hops = HOP_FLOPS * v * n
    if kind == "dirac":
        return {"bytes": 2 * n * field + links, "flops": hops}
    if kind in ("schur", "batch", "learned"):
        # about twenty applications of the reduced operator reach 1e-10 on these fields
        return {"bytes": 2 * n * coarse + links, "flops": 20 * hops}
    if kind == "drr":
        return {"bytes": 2 * n * field + links, "flops": 38 * hops}
    if kind == "approx":
        return {"bytes": 2 * n * coarse + links, "flops": 2 * hops}
    if kind == "grad":
        # per layer: eight transports of FIN colour vectors and the channel mixing, once forward, and
        # backward once for the inputs and once for the weights
        per = sum(8 * fi * 72 + 9 * fi * fo * 3 * 8 for fi, fo in zip(CHANNELS[:-1], CHANNELS[1:]))
        return {"bytes": 2 * n * field + links, "flops": 3 * per * v * n}
    return {"bytes": 2 * n * field + links, "flops": 52 * hops}


# ------------------------------------------------------------------ the same in 64 bits
class _Wilson:
    """D on fields (T, Z, Y, X, 3, 4, n), from the operator's definition."""

    def __init__(self, dims, links, m0, bc=BC):
        lx, ly, lz, lt = dims
        self.shape, self.d = (lt, lz, ly, lx), 4.0 + m0
        self.g = _gammas()
        self.u, self.ub = [], []
        for mu in range(4):
            ax = 3 - mu
            u = links[:, mu].reshape(self.shape + (3, 3)).clone()
            u.select(ax, dims[mu] - 1).mul_(bc[mu])
            self.u.append(u)
            self.ub.append(torch.roll(u, 1, ax).conj().transpose(-1, -2))

    def field(self, x):
        n = x.shape[0]
        return x.reshape((n,) + self.shape + (4, 3)).permute(1, 2, 3, 4, 6, 5, 0).contiguous()

    def flat(self, f):
        return f.permute(6, 0, 1, 2, 3, 5, 4).reshape(f.shape[-1], -1).contiguous()

    @staticmethod
    def colour(u, f):
        return torch.stack([sum(u[..., a, b, None, None] * f[..., b, :, :] for b in range(3)) for a in range(3)], -3)

    def spin(self, mu, f, sign):
        out = []
        for i in range(4):
            j = int(np.nonzero(self.g[mu, i])[0][0])
            out.append(f[..., i, :] + (sign * complex(self.g[mu, i, j])) * f[..., j, :])
        return torch.stack(out, -2)

    def __call__(self, f):
        out = self.d * f
        for mu in range(4):
            ax = 3 - mu
            out -= 0.5 * self.colour(self.u[mu], self.spin(mu, torch.roll(f, -1, ax), -1))
            out -= 0.5 * self.colour(self.ub[mu], self.spin(mu, torch.roll(f, 1, ax), 1))
        return out


def _solve(op, b, most=300):
    """BiCGstab per right-hand side (the last axis), to the rounding of 64 bits."""
    dims = tuple(range(b.dim() - 1))

    def dot(a, c):
        return (a.conj() * c).sum(dims)

    x = torch.zeros_like(b)
    r = b.clone()
    r0, p = r.clone(), r.clone()
    rho = dot(r0, r)
    bn = rho.real.clone()
    for _ in range(most):
        v = op(p)
        al = rho / dot(r0, v)
        s = r - al * v
        t = op(s)
        om = dot(t, s) / dot(t, t)
        x += al * p + om * s
        r = s - om * t
        if bool((dot(r, r).real <= 1e-28 * bn).all()):
            break
        rho2 = dot(r0, r)
        p = r + (rho2 / rho) * (al / om) * (p - om * v)
        rho = rho2
    return x


def _to_coarse(f, q, nb, w):
    n = f.shape[-1]
    site = w.flat(f).reshape(n, -1, 12)
    return site[:, torch.from_numpy(np.asarray(q[:nb], np.int64)).to(DEV)].reshape(n, -1)


def _from_coarse(x, q, nb, w, volume):
    n = x.shape[0]
    full = torch.zeros((n, volume, 12), dtype=torch.complex128, device=DEV)
    full[:, torch.from_numpy(np.asarray(q[:nb], np.int64)).to(DEV)] = x.reshape(n, nb, 12)
    return w.field(full.reshape(n, -1))


def _exact_schur(dims, m0, links, q, nb, x, approx=False):
    v = int(np.prod(dims))
    w = _Wilson(dims, links, m0)
    rest = (~_coarse_mask(q, nb, v)).reshape(w.shape + (1, 1, 1)).to(torch.float64)
    u = _from_coarse(x, q, nb, w, v)
    b = w(u) * rest
    if approx:
        rows = w(torch.ones(w.shape + (3, 4, 1), dtype=torch.complex128, device=DEV) * rest) * rest
        t = torch.where(rest > 0, b / torch.where(rest > 0, rows, 1.0), 0.0)
        z = (b - w(t) * rest) / w.d + t
    else:
        z = _solve(lambda p: w(p) * rest, b)
    return _to_coarse(w(u - z), q, nb, w)


def _exact_grad(case, d):
    """Loss and gradients with respect to the conjugate weights, by torch's own differentiation."""
    dims, n = d["dims"], case["nrhs"]
    w = _Wilson(dims, d["links"], case["m0"])
    rest = (~_coarse_mask(d["q"], d["nb"], d["V"])).reshape(w.shape + (1, 1, 1)).to(torch.float64)
    loss, ws = 0.0, [torch.from_numpy(a).to(DEV).requires_grad_() for a in _weights(case)]

    def mix(a, f):
        return torch.tensordot(f, a, dims=([5], [1])).movedim(-1, 5)

    def layer(f, a):
        out = mix(a[0], f)
        for mu in range(4):
            ax = 3 - mu
            out = out + mix(a[1 + 2 * mu], w.colour(w.u[mu], torch.roll(f, -1, ax)))
            out = out + mix(a[2 + 2 * mu], w.colour(w.ub[mu], torch.roll(f, 1, ax)))
        return out

    for i in range(n):
        f, e = w.field(d["x"][i:i + 1]), w.field(d["e"][i:i + 1])
        y = f
        for a in ws:
            y = layer(y, a)
        one = ((y * rest - e).abs().square().sum() / e.abs().square().sum()) / n
        one.backward()
        loss += float(one.detach())
    # torch's gradient of a real function is twice the derivative by the conjugate
    return {"loss": loss, "grad": torch.cat([a.grad.reshape(-1) / 2 for a in ws]).cpu().numpy()}


def exact(case, seed):
    kind = case["kind"]
    d = _inputs(case, seed)
    if kind == "batch":
        return torch.cat([_exact_schur(m["dims"], m["m0"], m["links"], m["q"], m["n_coarse"], x).reshape(-1)
                          for m, x in zip(d["members"], d["x"])])
    if kind in ("schur", "learned", "approx"):
        return _exact_schur(d["dims"], case["m0"], d["links"], d["q"], d["nb"], d["x"], kind == "approx")
    if kind == "grad":
        return _exact_grad(case, d)
    w = _Wilson(d["dims"], d["links"], case["m0"])
    f = w.field(d["x"])
    if kind == "dirac":
        return w.flat(w(f))
    if kind == "vcycle":
        return w.flat(_solve(w, f))
    rest = (~_coarse_mask(d["q"], d["nb"], d["V"])).reshape(w.shape + (1, 1, 1)).to(torch.float64)
    return w.flat(_solve(lambda p: w(p) * rest, f))
