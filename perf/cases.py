"""The work that programs have this library do, as measurable cases.

A case is one call (or one short sequence of calls) through the Python
binding on fields that are already on the GPU.  The kinds:

  dslash    out = D in or D^dag in                     Operator.apply_D / apply_Ddag
  sap       the SAP smoother                            Operator.sap_smooth (MR), _jacobi, _eo
  solve     D x = b from x = 0 to a relative residual   Operator.gcr_solve / bicgstab_solve
  train     forward and backward of the solve           CloverSolve (operator build, two solves, force)
  force     link gradient from two solutions            Operator.force
  setup     a new gauge field: build the operator,      Operator(...) and one apply_D
            then apply it once
  mg_setup  two-level hierarchy of one operator         Multigrid(...) and its export
  mg_apply  one application of that preconditioner      Multigrid.apply

Sizes, couplings and parameters are those of the benchmark, its side
measurements and the tests, or generic lattices of the same range (extents
that are multiples of 4, of 8 where the red/black colouring needs it).
"""
import math

import torch

from paper_2112_00501_amd import cloversap as cs

PREC = cs.PREC
SPINOR = {"f64": 192, "f32": 96, "f16": 52, "bf16": 52}     # bytes per site
LINKS = {"f64": 384, "f32": 192, "f16": 96, "bf16": 96}     # four links, rows 0 and 1
CLOVER = {"f64": 576, "f32": 288, "f16": 288, "bf16": 288}
FLOPS_D = 1944                                              # 8 hops of 168, the clover term, the sum
FLOPS_MR = 6 * 168 + 552 + 48 + 96 + 192                    # one MR step on the block operator


def _case(name, kind, dims, **more):
    c = dict(name=name, kind=kind, lx=dims[0], ly=dims[1], lz=dims[2], lt=dims[3], eps=0.3, kappa=0.1355, csw=1.0,
             antiperiodic=False)
    c.update(more)
    return c


def listed():
    return [
        # the smallest call there is in earnest: one operator application on the 8^4 lattice of
        # the smoke test, in double precision (the residual b - D x); launch latency
        _case("dslash_f64_8x8x8x8", "dslash", (8, 8, 8, 8), prec="f64", dagger=False, nrhs=1, kappa=0.13),
        # the operator of the benchmark lattice, far larger than the last-level cache
        _case("dslash_f32_32x32x32x64", "dslash", (32, 32, 32, 64), prec="f32", dagger=False, nrhs=1, eps=0.25,
              kappa=0.137, csw=1.1),
        # the adjoint in a 16-bit format on extents with odd block counts, a few right-hand sides,
        # antiperiodic time (the usual boundary condition of fermions)
        _case("ddag_f16_12x20x28x36_x3", "dslash", (12, 20, 28, 36), prec="f16", dagger=True, nrhs=3,
              antiperiodic=True),
        # the smoother as the benchmark's solver calls it: two cycles of four MR steps from zero
        _case("sap_f32_32x32x32x64", "sap", (32, 32, 32, 64), prec="f32", block="mr", n_cy=2, n_mr=4, zero=True,
              nrhs=1, eps=0.25, kappa=0.137, csw=1.1),
        # the smoother as a post-smoother: a start vector, a few right-hand sides, uneven extents
        _case("sap_bf16_8x24x40x16_x5", "sap", (8, 24, 40, 16), prec="bf16", block="mr", n_cy=1, n_mr=4, zero=False,
              nrhs=5, antiperiodic=True),
        # a propagator: the twelve spin-colour sources of a point in one batch
        _case("solve_x12_16x16x16x32", "solve", (16, 16, 16, 32), solver="gcr", inner="f32", basis="f32", block="mr",
              nrhs=12),
        # the benchmark's solve: one right-hand side, mixed precision, to 1e-10
        _case("solve_32x32x32x64", "solve", (32, 32, 32, 64), solver="gcr", inner="f32", basis="f32", block="mr",
              nrhs=1, eps=0.25, kappa=0.137, csw=1.1),
        # one training step through the differentiable solve
        _case("train_16x16x16x32", "train", (16, 16, 16, 32)),
        # the force alone (molecular dynamics: solutions in hand), double precision
        _case("force_24x24x24x48", "force", (24, 24, 24, 48)),
        # a new gauge field: operator build and its first application
        _case("setup_32x32x32x64", "setup", (32, 32, 32, 64), prec="f32"),
        # the multigrid hierarchy of a configuration, with the four adaptive passes of the paper
        _case("mg_setup_16x16x16x32", "mg_setup", (16, 16, 16, 32), nv=16, n_adapt=4),
        # one application of the multigrid preconditioner at the benchmark's size
        _case("mg_apply_32x32x32x64", "mg_apply", (32, 32, 32, 64), nv=16, n_adapt=1, eps=0.25, kappa=0.137, csw=1.1),
    ]


def _dims(rng, step, vmin, vmax):
    """Four extents, multiples of step, with the volume spread over its logarithm."""
    while True:
        side = math.exp(rng.uniform(math.log(vmin), math.log(vmax))) ** 0.25
        d = [step * max(1, round(side * rng.uniform(0.6, 1.6) / step)) for _ in range(4)]
        v = d[0] * d[1] * d[2] * d[3]
        if vmin <= v <= vmax:
            return d


def draw(rng):
    kind = rng.choice(["dslash", "dslash", "sap", "sap", "solve", "solve", "train", "force", "setup", "mg_setup",
                       "mg_apply"])
    big = 32 * 32 * 32 * 64
    step = 4 if kind in ("dslash", "force", "setup") else 8
    vmax = {"dslash": big, "sap": big, "solve": 16 * 16 * 24 * 32, "train": 16 * 16 * 16 * 32,
            "force": 24 * 24 * 24 * 48, "setup": big // 2, "mg_setup": 16 * 16 * 16 * 32, "mg_apply": big // 4}[kind]
    d = _dims(rng, step, 2048 if step == 4 else 4096, vmax)
    more = dict(antiperiodic=rng.random() < 0.5, kappa=rng.choice([0.13, 0.1355]))
    v = d[0] * d[1] * d[2] * d[3]
    if kind in ("dslash", "sap"):
        most = max(1, min(12, big // v))
        more.update(prec=rng.choice(["f64", "f32", "f16", "bf16"]), nrhs=rng.randint(1, most))
    if kind == "dslash":
        more.update(dagger=rng.random() < 0.5)
    elif kind == "sap":
        more.update(block=rng.choice(["mr", "mr", "jacobi", "eo"]), n_cy=rng.choice([1, 2]), n_mr=rng.choice([2, 4]),
                    zero=rng.random() < 0.7)
    elif kind == "solve":
        solver = rng.choice(["gcr", "gcr", "bicgstab"])
        inner = rng.choice(["f32", "f32", "f16", "bf16", "f64"])
        basis = "f64" if inner == "f64" else "f32"
        more.update(solver=solver, inner=inner, basis=basis, block=rng.choice(["mr", "mr", "jacobi", "eo"]),
                    nrhs=1 if solver == "bicgstab" else rng.choice([1, 2, 5, 12]))
    elif kind == "setup":
        more.update(prec=rng.choice(["f64", "f32"]))
    elif kind in ("mg_setup", "mg_apply"):
        more.update(nv=rng.choice([5, 8, 12, 16]), n_adapt=rng.choice([1, 2]))
    c = _case("", kind, d, **more)
    del c["name"]
    return c


# ------------------------------------------------------------------- inputs

def _geom(c):
    return c["lx"], c["ly"], c["lz"], c["lt"]


def _volume(c):
    return c["lx"] * c["ly"] * c["lz"] * c["lt"]


def _mm(a, b):
    return (a[..., :, :, None] * b[..., None, :, :]).sum(-2)


def _links(c, gen):
    """Links exp(i eps H), H Gaussian, Hermitian and traceless, put onto SU(3): complex128 [V][4][3][3]."""
    v = _volume(c)
    out = torch.empty((v * 4, 3, 3), dtype=torch.complex128, device="cuda")
    for s0 in range(0, v * 4, 1 << 21):
        n = min(v * 4, s0 + (1 << 21)) - s0
        r = torch.randn((n, 9), dtype=torch.float64, device="cuda", generator=gen)
        h = torch.zeros((n, 3, 3), dtype=torch.complex128, device="cuda")
        d = r[:, :3] - r[:, :3].mean(1, keepdim=True)
        for i in range(3):
            h[:, i, i] = d[:, i].to(torch.complex128)
        for j, (a, b) in enumerate(((0, 1), (0, 2), (1, 2))):
            z = torch.complex(r[:, 3 + 2 * j], r[:, 4 + 2 * j])
            h[:, a, b] = z
            h[:, b, a] = z.conj()
        a = (1j * c["eps"] / 8) * h
        eye = torch.eye(3, dtype=torch.complex128, device="cuda")
        u = eye + a / 6
        for k in range(5, 0, -1):
            u = eye + _mm(a, u) / k
        for _ in range(3):
            u = _mm(u, u)
        r0 = u[:, 0] / torch.linalg.vector_norm(u[:, 0], dim=-1, keepdim=True)
        r1 = u[:, 1] - (r0.conj() * u[:, 1]).sum(-1, keepdim=True) * r0
        r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
        out[s0:s0 + n, 0], out[s0:s0 + n, 1] = r0, r1
        out[s0:s0 + n, 2] = torch.linalg.cross(r0, r1).conj()
    return out.reshape(v, 4, 3, 3)


def _spinors(c, gen, n=1):
    v = _volume(c)
    r = torch.randn((n, v, 4, 3, 2), dtype=torch.float64, device="cuda", generator=gen)
    return torch.view_as_complex(r)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _params(c):
    return cs.SolverParams(inner_prec=PREC[c["inner"]], basis_prec=PREC[c["basis"]],
                           block_solver={"mr": 0, "jacobi": 1, "eo": 2}[c["block"]])


def _rhs(c, gen):
    """Right-hand sides and start vectors of a case, canonical complex128."""
    n = c.get("nrhs", 1)
    if c["kind"] == "sap" and not c["zero"]:
        return _spinors(c, gen, n), _spinors(c, gen, n)
    if c["kind"] in ("force", "train"):
        return _spinors(c, gen), _spinors(c, gen)
    return _spinors(c, gen, n), None


def prepare(case, seed):
    c, gen = case, _gen(seed)
    U = _links(c, gen)
    lat = cs.Lattice(_geom(c), antiperiodic_t=c["antiperiodic"])
    s = dict(case=c, lat=lat)
    kind = c["kind"]
    if kind == "train":
        b, g = _rhs(c, gen)
        s.update(U=U.requires_grad_(), b=b[0].requires_grad_(), g=g[0])
        return s
    if kind == "setup":
        b, _ = _rhs(c, gen)
        p = PREC[c["prec"]]
        s.update(U=U, b=lat.import_field(b, p), out=lat.new_field(p))
        return s
    op = s["op"] = cs.Operator(lat, U, c["kappa"], c["csw"])
    del U
    if kind in ("mg_setup", "mg_apply"):
        etas = lat.new_field(cs.F32, c["nv"])
        etas.view(torch.float32).normal_(generator=gen)
        params = cs.MgParams(nv=c["nv"], n_adapt=c["n_adapt"])
        if kind == "mg_setup":
            s.update(etas=etas, params=params)
            return s
        s["mg"] = cs.Multigrid(op, etas, params)
        s["b"] = lat.new_field(cs.F32)
        s["b"].view(torch.float32).normal_(generator=gen)
        s["x"] = lat.new_field(cs.F32)
        return s
    b, x = _rhs(c, gen)
    n = c.get("nrhs", 1)
    p = PREC[c["prec"]] if kind in ("dslash", "sap") else cs.F64
    s["b"] = lat.import_field(b, p)
    if x is not None:
        s["x0"] = lat.import_field(x, p)
    if kind == "force":
        return s
    s["x"] = lat.new_field(p, n)
    if kind == "solve":
        s["params"] = _params(c)
    return s


def _values(field, c, prec, nrhs):
    """The numbers of an internal-layout field: (mantissas, scales) per right-hand side for the 16-bit formats."""
    if prec == "f64":
        return field.view(torch.float64)
    if prec == "f32":
        return field.view(torch.float32)
    v = _volume(c)
    f = field.view(nrhs, v * 52)
    t = torch.float16 if prec == "f16" else torch.bfloat16
    return f[:, :v * 48].view(t), f[:, v * 48:].view(torch.float32)


def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "train":
        x = cs.CloverSolve.apply(s["U"], s["b"], s["lat"], c["kappa"], c["csw"])
        gU, gb = torch.autograd.grad(x, (s["U"], s["b"]), s["g"])
        return x.detach(), gU, gb
    if kind == "setup":
        op = cs.Operator(s["lat"], s["U"], c["kappa"], c["csw"])
        op.apply_D(s["out"], s["b"], PREC[c["prec"]])
        return _values(s["out"], c, c["prec"], 1)
    if kind == "force":
        return s["op"].force(s["b"], s["x0"], want_lie=True, want_grad=False)[0]
    if kind == "mg_setup":
        mg = cs.Multigrid(s["op"], s["etas"], s["params"])
        P, Dc = mg.export()
        return P.view(torch.float32), Dc
    if kind == "mg_apply":
        return s["mg"].apply(s["b"], s["x"]).view(torch.float32)
    op, n = s["op"], c["nrhs"]
    if kind == "dslash":
        f = op.apply_Ddag if c["dagger"] else op.apply_D
        f(s["x"], s["b"], PREC[c["prec"]], n)
        return _values(s["x"], c, c["prec"], n)
    if kind == "sap":
        f = {"mr": op.sap_smooth, "jacobi": op.sap_smooth_jacobi, "eo": op.sap_smooth_eo}[c["block"]]
        if not c["zero"]:
            s["x"].copy_(s["x0"])
        f(s["x"], s["b"], PREC[c["prec"]], c["n_cy"], c["n_mr"], c["zero"], n)
        return _values(s["x"], c, c["prec"], n)
    s["x"].zero_()
    if c["solver"] == "bicgstab":
        op.bicgstab_solve(s["x"], s["b"], s["params"])
    else:
        op.gcr_solve(s["x"], s["b"], s["params"], n)
    return s["x"].view(torch.float64)


# --------------------------------------------------------------------- work

def _sap_work(c, prec, n_cy, n_mr, zero):
    """Bytes per right-hand side and per operator, and flops, per site of one smoother call."""
    sp = SPINOR[prec]
    face = 2 * sp                         # two of the eight neighbours are outside the block
    rhs = op = fl = 0.0
    for cy in range(n_cy):
        for col in range(2):
            first = zero and cy == 0
            rhs += 0.5 * (2 * sp + (0 if first else sp) + (0 if first and col == 0 else face))
            op += 0.5 * (LINKS[prec] * (1.0 if first and col == 0 else 1.25) + CLOVER[prec])
            fl += 0.5 * (n_mr * FLOPS_MR + (0 if first and col == 0 else 336 if first else FLOPS_D))
    return rhs, op, fl


# outer iterations to 1e-10 by coupling, as measured on these lattices
_ITERS = {0.13: 14, 0.1355: 18, 0.137: 60}


def _solve_work(c, solver, inner, basis, nrhs):
    v, its = _volume(c), _ITERS[c["kappa"]]
    rhs, op, fl = _sap_work(c, inner, 2, 4, True)
    d_rhs, d_op = 2 * SPINOR[inner], LINKS[inner] + CLOVER[inner]
    # level 1 per iteration: the basis (eight vectors on average) read twice, w, r and its copy
    lev = 2 * 9 * SPINOR[basis] + 3 * 192 + SPINOR[inner]
    true = 3 * 192 + (LINKS["f64"] + CLOVER["f64"]) / nrhs
    per = rhs + d_rhs + (op + d_op) / nrhs + lev
    return v * nrhs * (its * per + 2 * true + 2 * 192), v * nrhs * (its * (fl + FLOPS_D + 16 * 12 * 9) + 2 * FLOPS_D)


def work(case):
    c, v, kind = case, _volume(case), case["kind"]
    if kind == "dslash":
        p, n = c["prec"], c["nrhs"]
        return dict(bytes=v * (2 * n * SPINOR[p] + LINKS[p] + CLOVER[p]), flops=v * n * FLOPS_D)
    if kind == "sap":
        rhs, op, fl = _sap_work(c, c["prec"], c["n_cy"], c["n_mr"], c["zero"])
        return dict(bytes=v * (c["nrhs"] * rhs + op), flops=v * c["nrhs"] * fl)
    build_b, build_f = 2304 / 4 + 384 + 576 + 288, 6 * 4 * 3 * 198.0
    if kind == "setup":
        p = c["prec"]
        return dict(bytes=v * (576 + 768 + 2 * 864 + 2 * SPINOR[p] + LINKS[p] + CLOVER[p]),
                    flops=v * (build_f + 2 * 1000 + FLOPS_D))
    if kind == "force":
        return dict(bytes=v * (2 * 192 + 384 + 4 * 64), flops=v * (4 * 12 * 3 * 198.0))
    if kind == "solve":
        b, f = _solve_work(c, c["solver"], c["inner"], c["basis"], c["nrhs"])
        return dict(bytes=b, flops=f)
    if kind == "train":
        b, f = _solve_work(c, "gcr", "f32", "f32", 1)
        return dict(bytes=2 * b + v * (build_b + 2 * 192 + 384 + 576), flops=2 * f + v * (build_f + 9504))
    nv, nblk = c["nv"], v // 256
    dc = nblk * 9 * (2 * nv) ** 2 * 8
    coarse_its = 10
    coarse = 2 * coarse_its * nblk * 5 * (2 * nv) ** 2 * 8
    rhs, op, fl = _sap_work(c, "f32", 2, 4, False)
    apply_b = v * (2 * (nv + 1) * 96 + rhs + op) + coarse
    apply_f = v * (2 * nv * 96 + fl) + coarse * 2
    if kind == "mg_apply":
        return dict(bytes=apply_b, flops=apply_f)
    rhs4, op4, fl4 = _sap_work(c, "f32", 4, 4, True)
    rebuild_b, rebuild_f = v * (2 * nv * 96 + 480) + dc, v * (2 * nv * FLOPS_D + 2 * (2 * nv) ** 2 * 48 + 8 * 12 * nv * nv)
    na = c["n_adapt"]
    return dict(bytes=v * (nv * rhs4 + op4) + (na + 1) * rebuild_b + na * (v * (nv * (4 * 96 + rhs) + op) + nv * coarse),
                flops=v * nv * fl4 + (na + 1) * rebuild_f + na * nv * apply_f)


# -------------------------------------------------- the same in plain torch

_DIM = (3, 2, 1, 0)  # array dimension of x, y, z, t in [t][z][y][x][...]


def _gammas():
    s = torch.tensor([[[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]]], dtype=torch.complex128)
    g = torch.zeros((4, 4, 4), dtype=torch.complex128)
    for k in range(3):
        g[k, :2, 2:], g[k, 2:, :2] = -1j * s[k], 1j * s[k]
    g[3, :2, 2:] = g[3, 2:, :2] = torch.eye(2)
    return g.cuda()


def _spin(m, psi):
    """A 4 x 4 matrix with few entries on the spins of psi[..., 4, 3]."""
    rows = []
    for i in range(4):
        acc = 0
        for j in range(4):
            z = complex(m[i, j])
            if z != 0:
                acc = acc + z * psi[..., j, :]
        rows.append(acc if torch.is_tensor(acc) else torch.zeros_like(psi[..., 0, :]))
    return torch.stack(rows, -2)


def _mv(u, psi):
    return (u[..., None, :, :] * psi[..., :, None, :]).sum(-1)


class _Exact:
    """The operator of one case in double precision on [t][z][y][x] arrays."""

    def __init__(self, c, U):
        lx, ly, lz, lt = _geom(c)
        self.c, self.kappa = c, c["kappa"]
        self.shape = (lt, lz, ly, lx)
        self.gam = _gammas().cpu()
        self.g5 = torch.diag(torch.tensor([1, 1, -1, -1], dtype=torch.complex128))
        u = U.reshape(*self.shape, 4, 3, 3)
        self.u = [u[..., m, :, :] for m in range(4)]
        self.hop = list(self.u)
        if c["antiperiodic"]:
            s = torch.ones((lt, 1, 1, 1, 1, 1), dtype=torch.float64, device=U.device)
            s[-1] = -1
            self.hop[3] = self.u[3] * s
        self.one = torch.eye(4, dtype=torch.complex128)
        self.planes = [(m, n) for m in range(4) for n in range(m + 1, 4)]
        self.F = [self._field(m, n) for m, n in self.planes]
        self.sig = [0.5j * (self.gam[m] @ self.gam[n] - self.gam[n] @ self.gam[m]) for m, n in self.planes]

    def _field(self, m, n):
        dag = lambda a: a.conj().transpose(-1, -2)  # noqa: E731
        sh = lambda a, d, k: torch.roll(a, -k, _DIM[d])  # noqa: E731  a(x + k d)
        um, un = self.u[m], self.u[n]
        plaq = _mm(_mm(um, sh(un, m, 1)), dag(_mm(un, sh(um, n, 1))))              # from x: m, n, -m, -n
        ph = _mm(_mm(un, dag(sh(sh(um, m, -1), n, 1))), _mm(dag(sh(un, m, -1)), sh(um, m, -1)))
        q = plaq + ph
        a, b = sh(um, m, -1), sh(sh(un, m, -1), n, -1)
        q = q + _mm(_mm(dag(a), dag(b)), _mm(sh(sh(um, m, -1), n, -1), sh(un, n, -1)))
        q = q + _mm(_mm(dag(sh(un, n, -1)), sh(um, n, -1)), _mm(sh(sh(un, n, -1), m, 1), dag(um)))
        return (q - dag(q)) / 8

    def clover(self, psi):
        out = psi
        for f, s in zip(self.F, self.sig):
            out = out + (1j * self.kappa * self.c["csw"]) * _spin(s, _mv(f, psi))
        return out

    def hops(self, psi, inside=None):
        """Hopping sum; inside: only hops within the 4^4 blocks."""
        acc = 0
        for m in range(4):
            d = _DIM[m]
            up = torch.roll(_spin(self.one, psi), -1, d)
            t = _mv(self.hop[m], _spin(self.one - self.gam[m], up))
            w = torch.roll(_mv(self.hop[m].conj().transpose(-1, -2), _spin(self.one + self.gam[m], psi)), 1, d)
            if inside is not None:
                i = torch.arange(self.shape[d], device=psi.device) % 4
                view = [1] * 6
                view[d] = -1
                t = t * (i != 3).view(view)
                w = w * (i != 0).view(view)
            acc = acc + t + w
        return acc

    def D(self, psi):
        return self.clover(psi) - self.kappa * self.hops(psi)

    def DB(self, psi):
        return self.clover(psi) - self.kappa * self.hops(psi, True)

    # ---- SAP
    def _blocks(self, a):
        lt, lz, ly, lx = self.shape
        a = a.reshape(lt // 4, 4, lz // 4, 4, ly // 4, 4, lx // 4, 4, -1).sum((1, 3, 5, 7, 8))
        for d in range(4):
            a = a.repeat_interleave(4, d)
        return a[..., None, None]

    def cinv(self):
        """(1 + T)^-1 as matrices [..., 12, 12]."""
        e = torch.eye(12, dtype=torch.complex128, device=self.F[0].device).reshape(12, 4, 3)
        cols = [self.clover(e[k].expand(*self.shape, 4, 3)).reshape(*self.shape, 12) for k in range(12)]
        return torch.linalg.inv(torch.stack(cols, -1))

    def sap(self, x, b, block, n_cy, n_mr):
        lt, lz, ly, lx = self.shape
        idx = [torch.arange(n, device=b.device) for n in self.shape]
        par = sum((i // 4).view([-1 if d == k else 1 for k in range(4)]) for d, i in enumerate(idx)) % 2
        site = sum(i.view([-1 if d == k else 1 for k in range(4)]) for d, i in enumerate(idx)) % 2
        even = (site == 0)[..., None, None]
        if block != "mr":
            ci = self.cinv()
            C = lambda v: (ci * v.reshape(*self.shape, 1, 12)).sum(-1).reshape(v.shape)  # noqa: E731

        def mr(op, r, steps):
            delta = torch.zeros_like(r)
            for _ in range(steps):
                q = op(r)
                qq = self._blocks(q.real ** 2 + q.imag ** 2)
                a = self._blocks(q.conj() * r) / torch.where(qq > 0, qq, 1.0)
                delta = delta + a * r
                r = r - a * q
            return delta

        for _ in range(n_cy):
            for col in range(2):
                mask = (par == col)[..., None, None]
                r = (b - self.D(x)) * mask
                if block == "mr":
                    d = mr(self.DB, r, n_mr)
                elif block == "jacobi":
                    rho = C(r)
                    d = torch.zeros_like(r)
                    for _ in range(n_mr):
                        d = rho + self.kappa * C(self.hops(d, True))
                else:
                    k = self.kappa
                    S = lambda v: (self.clover(v) - k * k * self.hops(C(self.hops(v, True) * ~even), True)) * even  # noqa: E731
                    d = mr(S, (r + k * self.hops(C(r * ~even), True)) * even, n_mr)
                    d = d + C((r + k * self.hops(d, True)) * ~even)
                x = x + d * mask
        return x

    # ---- solve: BiCGStab restarted from the true residual until it no longer falls
    def solve(self, b):
        x = torch.zeros_like(b)
        bn = float(torch.linalg.vector_norm(b))
        last = math.inf
        for _ in range(12):
            r = b - self.D(x)
            rn = float(torch.linalg.vector_norm(r))
            if rn < 3e-15 * bn or rn > 0.5 * last:
                break
            last = rn
            rh, p, v = r.clone(), torch.zeros_like(r), torch.zeros_like(r)
            rho = al = om = 1.0
            for _ in range(600):
                rho1 = complex(torch.vdot(rh.reshape(-1), r.reshape(-1)))
                p = r + (rho1 / rho) * (al / om) * (p - om * v)
                rho = rho1
                v = self.D(p)
                al = rho / complex(torch.vdot(rh.reshape(-1), v.reshape(-1)))
                s = r - al * v
                t = self.D(s)
                om = complex(torch.vdot(t.reshape(-1), s.reshape(-1)) / torch.vdot(t.reshape(-1), t.reshape(-1)).real)
                x = x + al * p + om * s
                r = s - om * t
                if float(torch.linalg.vector_norm(r)) < 1e-6 * rn:
                    break
        return x

    def dag_solve(self, b):
        return _spin(self.g5, self.solve(_spin(self.g5, b)))


def _lie(c, U, x, y):
    """g[site][mu][a] = dL/dw for dL = -Re(y^dag dD x), U -> exp(i w T^a) U."""
    U = U.detach().clone().requires_grad_()
    e = _Exact(c, U)
    (-(y.conj() * e.D(x)).sum().real).backward()
    G = U.grad.reshape(-1, 4, 3, 3)
    U = U.detach().reshape(-1, 4, 3, 3)
    M = _mm(U, G.conj().transpose(-1, -2))              # g_a = Re tr(G^dag i T^a U)
    out = []
    for T in _generators():
        out.append((1j * (T.cuda() * M.transpose(-1, -2)).sum((-1, -2))).real)
    return torch.stack(out, -1)


def _generators():
    g = torch.zeros((8, 3, 3), dtype=torch.complex128)
    for n, (a, b) in zip((0, 3, 5), ((0, 1), (0, 2), (1, 2))):
        g[n, a, b] = g[n, b, a] = 0.5
        g[n + 1, a, b], g[n + 1, b, a] = -0.5j, 0.5j
    # the order 1..8 of Gell-Mann: 1, 2 (01), 3 (diagonal), 4, 5 (02), 6, 7 (12), 8 (diagonal)
    out = torch.stack([g[0], g[1], torch.diag(torch.tensor([0.5, -0.5, 0], dtype=torch.complex128)), g[3], g[4], g[5],
                       g[6], torch.diag(torch.tensor([1, 1, -2], dtype=torch.complex128)) / (2 * math.sqrt(3))])
    return out


def _internal(c, psi, prec):
    """Canonical fields [n][V][4][3] (or [t][z][y][x] arrays) as the numbers of the internal layout."""
    lx, ly, lz, lt = _geom(c)
    n = psi.numel() // (_volume(c) * 12)
    a = psi.reshape(n, lt // 4, 4, lz // 4, 4, ly // 4, 4, lx // 4, 4, 12)
    a = a.permute(0, 1, 3, 5, 7, 2, 4, 6, 8, 9).reshape(n, -1, 256, 12)       # [n][block][site][component]
    r = torch.view_as_real(a.contiguous())                                     # ... [2]
    nblk = r.shape[1]
    if prec == "f64":
        return r.permute(0, 1, 3, 2, 4).reshape(-1)
    if prec == "f32":
        return r.reshape(n, nblk, 256, 6, 4).permute(0, 1, 3, 2, 4).reshape(-1)
    scale = r.abs().amax((-1, -2))
    m = r / scale.clamp_min(1e-300)[..., None, None]
    return (m.reshape(n, nblk, 256, 3, 8).permute(0, 1, 3, 2, 4).reshape(n, -1), scale.reshape(n, -1))


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("mg_setup", "mg_apply"):
        return None  # the hierarchy follows from many single-precision steps
    n = c.get("nrhs", 1)
    if kind == "solve" and _volume(c) * n * _ITERS[c["kappa"]] > 16 * 16 * 16 * 32 * 13 * 18:
        return None  # takes too long
    gen = _gen(seed)
    U = _links(c, gen)
    b, x0 = _rhs(c, gen)
    shape = (c["lt"], c["lz"], c["ly"], c["lx"], 4, 3)
    if kind == "force":
        return _lie(c, U, b[0].reshape(shape), x0[0].reshape(shape)).reshape(_volume(c), 4, 8)
    e = _Exact(c, U)
    if kind == "train":
        x = e.solve(b[0].reshape(shape))
        y = e.dag_solve(x0[0].reshape(shape))
        g = _lie(c, U, x, y)
        P = sum(g[..., a, None, None] * T.cuda() for a, T in enumerate(_generators()))
        v = _volume(c)
        return x.reshape(v, 4, 3), _mm(2j * P, U), y.reshape(v, 4, 3)
    out = []
    for j in range(n):
        bj = b[j].reshape(shape)
        if kind == "dslash" and c["dagger"]:
            out.append(_spin(e.g5, e.D(_spin(e.g5, bj))))
        elif kind in ("dslash", "setup"):
            out.append(e.D(bj))
        elif kind == "sap":
            out.append(e.sap(torch.zeros_like(bj) if c["zero"] else x0[j].reshape(shape), bj, c["block"], c["n_cy"],
                             c["n_mr"]))
        else:
            out.append(e.solve(bj))
    return _internal(c, torch.stack(out), c.get("prec", "f64"))
