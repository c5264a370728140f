"""The workloads this library is timed on: what its users run, by its public calls.

Every case is a plain dict: the call (`kind`), the lattice, whether the operator has
long links, the number of right-hand sides, and for the solvers the storage precision,
the mass and the tolerance.

  apply   Context.apply: A x in FP64 (measurement codes, preconditioners, checks)
  solve   Context.solve: blockCGrQ, the main call
  cg      Context.solve_cg: the single right-hand-side solver
  pseudo  Context.solve_pseudo: N recurrences sharing the stencil (FP64 storage)
  force   Context.link_force: the gradients with respect to the links
  grad    BlockSolve forward and backward of L = Re sum_i b_i^H A^{-1} b_i

Inputs follow the distributions of paper_1710_09745_amd.synth (Gaussian fat links,
Haar SU(3) long links, Gaussian right-hand sides), drawn on the GPU from the seed.
"""
import math

import torch

from paper_1710_09745_amd import bcg

DEV = "cuda"

# Reference solves that would take longer than this estimate (site-columns times
# iterations) have no 64-bit reference here.
EXACT_WORK_LIMIT = 8.0e9


def _case(name, kind, dims, improved, nrhs, prec="fp64", mass=0.0, tol=0.0):
    c = {"name": name, "kind": kind, "improved": improved, "nrhs": nrhs, "prec": prec, "mass": mass, "tol": tol}
    c.update(zip(("lx", "ly", "lz", "lt"), dims))
    return c


def listed():
    return [
        # the smallest calls: a naive 4^4 operator with four columns, where launches count
        _case("apply_4x4x4x4_naive_n4", "apply", (4, 4, 4, 4), False, 4, mass=0.1),
        _case("solve_4x4x4x4_naive_n4", "solve", (4, 4, 4, 4), False, 4, "fp64", 0.1, 1e-10),
        # the headline lattice of bench.py: operator and FP64 block solve
        _case("apply_16x16x16x16_n16", "apply", (16, 16, 16, 16), True, 16, mass=0.05),
        _case("solve_16x16x16x16_n16_fp64", "solve", (16, 16, 16, 16), True, 16, "fp64", 0.05, 1e-10),
        # a ragged column count on the largest lattice, beyond every cache
        _case("apply_32x32x32x64_n12", "apply", (32, 32, 32, 64), True, 12, mass=0.02),
        # the diluted-source workload's lattice: 32 sources at a time
        _case("solve_16x16x16x48_n32_fp32", "solve", (16, 16, 16, 48), True, 32, "fp32", 0.05, 1e-10),
        # 16-bit fixed-point storage on a lattice that is no power of two
        _case("solve_24x24x24x24_n24_fix16", "solve", (24, 24, 24, 24), True, 24, "fix16", 0.05, 1e-10),
        # the largest solve: FP32 storage with FP64 reliable updates (a heavier mass than
        # bench.py's keeps a pass near a second)
        _case("solve_32x32x32x64_n16_fp32", "solve", (32, 32, 32, 64), True, 16, "fp32", 0.1, 1e-10),
        # one right-hand side: conjugate gradient in FP32 storage with FP64 updates
        _case("cg_32x32x32x64_n1_fp32", "cg", (32, 32, 32, 64), True, 1, "fp32", 0.1, 1e-10),
        # pseudo-block CG at a block size that is no power of two
        _case("pseudo_16x16x16x48_n24_fp64", "pseudo", (16, 16, 16, 48), True, 24, "fp64", 0.05, 1e-10),
        # training through the solve: forward, adjoint solve and link force
        _case("grad_16x16x16x16_n8_fp64", "grad", (16, 16, 16, 16), True, 8, "fp64", 0.05, 1e-10),
        # the link force alone, as a molecular-dynamics step with its solutions in hand calls it
        _case("force_16x16x16x48_n16", "force", (16, 16, 16, 48), True, 16, mass=0.05),
    ]


def _volume(case):
    return case["lx"] * case["ly"] * case["lz"] * case["lt"]


def _dims(case):
    return (case["lx"], case["ly"], case["lz"], case["lt"])


def _iterations(case):
    """Iterations of a conjugate-gradient type solve from the condition number: the
    largest eigenvalue of A is near 50 with long links (839 iterations were seen at
    m = 0.05, 1e-10) and near 16 without, the smallest is 4 m^2."""
    root_lmax = 7.1 if case["improved"] else 4.0
    return max(1.0, 0.25 * root_lmax / case["mass"] * math.log(2.0 / case["tol"]))


def _cost(case):
    """Relative time of a pass: bytes moved, with each site's links and a launch floor."""
    nl = 16 if case["improved"] else 8
    lm, vc = {"fp64": (144, 16.0), "fp32": (72, 8.0), "fix16": (40, 16.0 / 3.0)}[case["prec"]]
    site = nl * lm * 2 + case["nrhs"] * (60 * vc + 96) * max(1.0, case["nrhs"] / 16.0)
    it = _iterations(case) if case["kind"] in ("solve", "cg", "pseudo", "grad") else 1.0
    if case["kind"] == "grad":
        it *= 2.0
    if case["kind"] == "cg":
        it *= case["nrhs"]
    return it * max(site * _volume(case) / 2, 4.0e7)


def draw(rng):
    """One more case: lattices from 4^4 to 32^3 x 64 with even extents of any kind, 1 to
    64 columns, both operators, and every storage precision that converges reliably."""
    limit = max(_cost(c) for c in listed())
    while True:
        kind = rng.choices(("apply", "solve", "cg", "pseudo", "force", "grad"), (6, 9, 1, 2, 2, 2))[0]
        target = 2.0 ** rng.uniform(8.0, 21.0)
        shape = [rng.uniform(0.75, 1.35) for _ in range(4)]
        scale = (target / math.prod(shape)) ** 0.25
        dims = tuple(min(64, max(4, 2 * round(s * scale / 2))) for s in shape)
        rows = 3 * math.prod(dims) // 2
        n = min(64, int(2.0 ** rng.uniform(0.0, 6.05)))
        if n < 1 or 96 * n > rows:
            continue
        if kind == "cg":
            n = rng.choice((1, 1, 2))
        prec, mass, tol = "fp64", rng.choice((0.02, 0.05, 0.1)), 0.0
        if kind in ("solve", "cg"):
            prec = rng.choice(("fp64", "fp64", "fp32", "fp32", "fix16") if kind == "solve" else ("fp64", "fp32"))
        if kind in ("solve", "cg", "pseudo", "grad"):
            mass, tol = rng.choice((0.05, 0.07, 0.1, 0.15)), 1e-10
        case = _case("", kind, dims, rng.random() < 0.85, n, prec, mass, tol)
        del case["name"]
        if math.prod(dims) <= 32 * 32 * 32 * 64 and _cost(case) <= limit:
            return case


# -- inputs ---------------------------------------------------------------------------------------
def _complex_normal(gen, shape, scale=1.0):
    x = torch.randn(*shape, 2, dtype=torch.float64, device=DEV, generator=gen)
    return torch.view_as_complex(x) * scale


def _haar_su3(gen, shape):
    """Haar SU(3): two Gaussian rows made orthonormal, the third their conjugate cross product."""
    a = _complex_normal(gen, (*shape, 3))
    a = a / torch.linalg.vector_norm(a, dim=-1, keepdim=True)
    b = _complex_normal(gen, (*shape, 3))
    b = b - (a.conj() * b).sum(-1, keepdim=True) * a
    b = b / torch.linalg.vector_norm(b, dim=-1, keepdim=True)
    return torch.stack((a, b, torch.linalg.cross(a, b).conj()), dim=-2).contiguous()


def _inputs(case, seed):
    """Links, and the right-hand sides (force: the pair X, Lambda)."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    v = _volume(case)
    if case["improved"]:
        fat = _complex_normal(gen, (4, v, 3, 3), 1.0 / 3.0)
        lng = _haar_su3(gen, (4, v))
    else:
        fat, lng = _haar_su3(gen, (4, v)), None
    vectors = [_complex_normal(gen, (case["nrhs"], v // 2, 3)) for _ in range(2 if case["kind"] == "force" else 1)]
    return fat, lng, vectors


def prepare(case, seed):
    """A context with its links, mass and solver settings, and the vectors on the GPU."""
    fat, lng, vectors = _inputs(case, seed)
    ctx = bcg.Context(_dims(case), improved=case["improved"])
    ctx.load_links(fat, lng)
    ctx.set_mass(case["mass"])
    if case["tol"]:
        ctx.set_solver(tol=case["tol"], max_iter=20000, prec=case["prec"], ru_delta=0.1)
    state = {"kind": case["kind"], "ctx": ctx, "vectors": vectors}
    if case["kind"] == "grad":
        state["fat"], state["lng"] = fat.requires_grad_(), None if lng is None else lng.requires_grad_()
        vectors[0].requires_grad_()
    return state


def run(state):
    kind, ctx = state["kind"], state["ctx"]
    if kind == "apply":
        return ctx.apply(state["vectors"][0])
    if kind == "solve":
        return ctx.solve(state["vectors"][0])[0]
    if kind == "cg":
        return ctx.solve_cg(state["vectors"][0])[0]
    if kind == "pseudo":
        return ctx.solve_pseudo(state["vectors"][0])[0]
    if kind == "force":
        fat, lng = ctx.link_force(*state["vectors"])
        return {"fat": fat} if lng is None else {"fat": fat, "long": lng}
    b, fat, lng = state["vectors"][0], state["fat"], state["lng"]
    x = bcg.BlockSolve.apply(b, fat, lng, ctx)
    loss = (b.conj() * x).sum().real
    wrt = [b, fat] if lng is None else [b, fat, lng]
    grads = torch.autograd.grad(loss, wrt)
    return {"x": x.detach(), "grads": list(grads)}


# -- what a pass cannot do without ----------------------------------------------------------------
def work(case):
    """apply, force: every link (both parities share them) and vector read once, every
    result written once.  Solvers: per iteration, both hops stream the links of their
    output parity, and the block vectors are read and written once in each of the
    passes that the recurrence's reductions separate."""
    vh, n, nl = _volume(case) // 2, case["nrhs"], 16 if case["improved"] else 8
    lm, vc = {"fp64": (144, 16.0), "fp32": (72, 8.0), "fix16": (40, 16.0 / 3.0)}[case["prec"]]
    hops = 2 * nl * 72 * n * vh
    if case["kind"] == "apply":
        return {"bytes": nl * 144 * vh + 96 * n * vh, "flops": hops}
    if case["kind"] == "force":
        return {"bytes": nl * 144 * vh + nl * 144 * vh + 96 * n * vh, "flops": 2 * hops + nl * 72 * n * 2 * vh}
    it = _iterations(case)
    if case["kind"] in ("solve", "grad"):
        # hops 6 + 9, pass A 9, pass B 12 + the FP64 X; the N x N products as complex flops
        site = 2 * nl * lm + 36 * n * vc + 96 * n
        flops = hops + 3 * 8 * n * n * 5 * vh
    else:
        # hops 6 + 9, X and R updates 18, P update 9
        site = 2 * nl * lm + 42 * n * vc
        flops = hops + 3 * 8 * n * 5 * vh
        if case["kind"] == "cg":
            site, flops = site + (n - 1) * 2 * nl * lm, flops
    times = it * (2 if case["kind"] == "grad" else 1)
    return {"bytes": times * site * vh, "flops": times * flops}


# -- the same results in plain torch, 64 bits -----------------------------------------------------
class _Plain:
    """A = 4 m^2 - D_eo D_oe on [V/2, 3, N] fields, from its definition."""

    def __init__(self, case, fat, lng):
        lx, ly, lz, lt = self.dims = _dims(case)
        self.mass, v = case["mass"], _volume(case)
        self.stride = (1, lx, lx * ly, lx * ly * lz)
        lex = torch.arange(v, device=DEV)
        x = torch.stack((lex % lx, lex // lx % ly, lex // (lx * ly) % lz, lex // (lx * ly * lz)))
        odd = x.sum(0) % 2
        self.sites = [lex[odd == p] for p in (0, 1)]
        self.x = [x[:, s] for s in self.sites]
        self.links = [(1, fat)] + ([] if lng is None else [(3, lng)])

    def eta(self, p, mu):
        return (1 - 2 * (self.x[p][:mu].sum(0) % 2)).double()

    def step(self, p, mu, d):
        """Full-lattice index of x + d mu for the sites of parity p."""
        x, size = self.x[p][mu], self.dims[mu]
        return self.sites[p] + ((x + d) % size - x) * self.stride[mu]

    def hop(self, p, v):
        out = torch.zeros_like(v)
        for mu in range(4):
            eta = self.eta(p, mu)[:, None, None]
            for length, u in self.links:
                ahead, behind = self.step(p, mu, length), self.step(p, mu, -length)
                for w, near in ((u[mu, self.sites[p]] * eta, ahead), (u[mu, behind].mH * -eta, behind)):
                    near = v[near >> 1]
                    for b in range(3):
                        out.addcmul_(w[:, :, b : b + 1], near[:, b : b + 1, :])
        return out

    def apply(self, v):
        return 4 * self.mass**2 * v - self.hop(0, self.hop(1, v))

    def solve(self, b, iterations):
        """Conjugate gradients on every column, as far as 64 bits go."""
        x = torch.zeros_like(b)
        for _ in range(2):
            r = b - self.apply(x)
            p, rr = r.clone(), (r.abs() ** 2).sum((0, 1))
            for k in range(iterations):
                ap = self.apply(p)
                alpha = rr / (p.conj() * ap).sum((0, 1)).real
                x += alpha * p
                r -= alpha * ap
                new = (r.abs() ** 2).sum((0, 1))
                p = r + (new / rr) * p
                rr = new
                if k % 32 == 31 and (rr / (b.abs() ** 2).sum((0, 1))).max() < 1e-27:
                    break
        return x

    def force(self, x, lam):
        yx, yl = self.hop(1, x), self.hop(1, lam)
        grads = []
        for length, u in self.links:
            g = torch.empty_like(u)
            for mu in range(4):
                for p, (u1, v1, u2, v2) in enumerate(((lam, yx, x, yl), (yx, lam, yl, x))):
                    near = self.step(p, mu, length) >> 1
                    s = self.eta(p, mu)[:, None] * (1 - 2 * p)
                    for a in range(3):
                        for c in range(3):
                            prod = (u1[:, a] * v1[near, c].conj() + u2[:, a] * v2[near, c].conj()).sum(-1, keepdim=True)
                            g[mu, self.sites[p], a, c] = (s * prod)[:, 0]
            grads.append(g)
        return grads


def _inner(v):
    return v.permute(1, 2, 0).contiguous()


def _outer(v):
    return v.permute(2, 0, 1).contiguous()


def exact(case, seed):
    fat, lng, vectors = _inputs(case, seed)
    plain = _Plain(case, fat, lng)
    kind = case["kind"]
    if kind == "apply":
        return torch.cat([_outer(plain.apply(_inner(v))) for v in vectors[0].split(4)])
    if kind == "force":
        g = plain.force(_inner(vectors[0]), _inner(vectors[1]))
        return {"fat": g[0]} if lng is None else {"fat": g[0], "long": g[1]}
    iterations = 40 + int(1.5 * _iterations(dict(case, tol=1e-13)))
    if (_volume(case) // 2) * (case["nrhs"] + 4) * iterations > EXACT_WORK_LIMIT:
        return None
    b = _inner(vectors[0])
    x = plain.solve(b, iterations)
    if kind != "grad":
        return _outer(x)
    # L = Re b^H A^{-1} b: dL/dX = b, so the adjoint solution is X itself
    return {"x": _outer(x), "grads": [_outer(2 * x)] + plain.force(x, x)}
