"""The workloads by which this framework's speed is followed.

Each case is one call, or one short sequence of calls, of the public Python
entry points, at the sizes of the repository's workloads (2D convection-
diffusion 1023^2 on 32 slabs, 2D Poisson 127^2 on 8, 2D Helmholtz with 64
slabs, 3D variable coefficient, the interface GMRES of the 3D Poisson tables)
and at ragged sizes between them.

  listed()   the cases followed by name
  draw(rng)  one more case of the same ranges
  prepare    the inputs (from the seed) and what a program keeps between calls
  run        one pass through the entry points
  work       bytes and operations that the path cannot do without
  exact      the same outputs by plain torch in FP64
"""
from __future__ import annotations

import itertools
import math

import torch

from paper_2510_25991_amd import ddst

DEV = "cuda"
F64 = torch.float64


# ---------------------------------------------------------------- cases
def _case(kind, dim, n, slabs, pde, precision, **kw):
    c = {"kind": kind, "dim": dim, "n": n, "slabs": slabs, "pde": pde, "precision": precision}
    c.update(kw)
    return c


def listed():
    return [
        # a product with the equilibrium matrix and one with its transpose, as
        # a serving loop calls them: nothing but latency
        _case("apply", 2, 255, 8, "diffusion", "fp64", name="diffusion2d_255_fp64_apply"),
        # a small problem solved once, set-up included: launches and the
        # serial chain of the eliminations
        _case("step", 2, 127, 8, "poisson", "fp64", name="poisson2d_127_fp64_step"),
        # the repository's headline: build + refined solve, mixed precision
        _case("step", 2, 1023, 32, "convdiff", "fp32", name="convdiff2d_1023_fp32_step"),
        # the same in plain FP64 on a ragged grid (M = 899, 30 planes a slab)
        _case("step", 2, 899, 30, "convdiff", "fp64", name="convdiff2d_899_fp64_step"),
        # time stepping: one more load with a kept operator
        _case("solve", 2, 1023, 32, "convdiff", "fp32", nrhs=1, name="convdiff2d_1023_fp32_solve"),
        # eight loads at once with a kept operator
        _case("solve", 2, 1023, 32, "convdiff", "fp32", nrhs=8, name="convdiff2d_1023_fp32_many8"),
        # one iteration of a coefficient inversion: differentiable solve,
        # sensor loss, gradients for kappa and the load
        _case("train", 2, 767, 24, "convdiff", "fp32", name="convdiff2d_767_fp32_train"),
        # 3D variable coefficient, symmetric elimination, one node more than
        # a multiple of 128 per interface (M = 3969)
        _case("step", 3, 63, 8, "diffusion", "fp32", name="diffusion3d_63_fp32_step"),
        # long Krylov runs: oscillatory problem, compressed blocks
        _case("hodlr", 2, 1023, 64, "helmholtz", "fp32", k=60.0, name="helmholtz2d_1023_hodlr_solve"),
        # the sampled route end to end: set-up without blocks, HBS from
        # samples, solve with the FP32 Krylov basis
        _case("sampled", 2, 511, 32, "helmholtz", "fp32", k=30.0, name="helmholtz2d_511_sampled"),
        # compression alone, then a product with the compressed form
        _case("compress", 2, 639, 20, "convdiff", "fp64", name="convdiff2d_639_fp64_compress"),
        # the interface system of the 3D Poisson tables (N = 32^3, H = 1/8)
        _case("gmres", 3, 31, 8, "poisson", "fp64", name="poisson3d_31_fp64_gmres"),
    ]


def draw(rng):
    """Sizes: slabs of 4..32 cells, 4..32 slabs, at most 1023 nodes per axis in
    2D and 63 in 3D, n + 1 spread over its logarithm."""
    kind = rng.choice(["step", "step", "step", "solve", "solve", "train", "hodlr", "sampled",
                       "compress", "gmres", "apply"])
    dim = 3 if kind == "gmres" or (kind in ("step", "solve", "train") and rng.random() < 0.3) else 2
    lo, hi = (32, 1024) if dim == 2 else (16, 64 if kind != "gmres" else 40)
    if kind in ("hodlr", "sampled", "compress"):
        lo, hi = 192, 768
    while True:
        want = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        slabs = rng.randint(4, 32 if dim == 2 else 8)
        m = round(want / slabs)
        if 4 <= m <= 32 and lo <= m * slabs <= hi:
            break
    n = m * slabs - 1
    if kind in ("hodlr", "sampled"):
        return _case(kind, 2, n, slabs, "helmholtz", "fp32", k=0.5 * slabs)
    pde = "poisson" if kind == "gmres" else rng.choice(["convdiff", "convdiff", "diffusion", "poisson"])
    precision = "fp64" if kind in ("compress", "gmres", "apply") else rng.choice(["fp32", "fp32", "fp64"])
    if kind == "train" and pde == "poisson":
        pde = "diffusion"
    case = _case(kind, dim, n, slabs, pde, precision)
    if kind == "solve":
        case["nrhs"] = rng.choice([1, 1, 2, 5, 8, 16])
    return case


# ---------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _fourier(dim, cells, seed, modes, kmax):
    """sum xi / |k|^2 cos(2 pi k.x + phi) at the cell centres (the spectrum of
    the variable-coefficient workloads)."""
    cpu = torch.Generator()
    cpu.manual_seed(int(seed))
    ks = [k for k in itertools.product(range(-kmax, kmax + 1), repeat=dim)
          if 0 < sum(v * v for v in k) <= kmax * kmax and next(v for v in k if v) > 0]
    pick = torch.randperm(len(ks), generator=cpu)[:modes].tolist()
    amp = torch.randn(modes, generator=cpu, dtype=F64).tolist()
    phase = (2 * math.pi * torch.rand(modes, generator=cpu, dtype=F64)).tolist()
    x = (torch.arange(cells, device=DEV, dtype=F64) + 0.5) / cells
    grid = [x.reshape([-1 if a == b else 1 for b in range(dim)]) for a in range(dim)]
    out = torch.zeros((cells,) * dim, device=DEV, dtype=F64)
    for i, a, ph in zip(pick, amp, phase):
        k = ks[i]
        arg = sum(2 * math.pi * k[d] * grid[d] for d in range(dim)) + ph
        out += a / float(sum(v * v for v in k)) * torch.cos(arg)
    return out


def _problem(case, seed):
    """Coefficients of the operator: kappa, velocity, zeroth-order term."""
    dim, n, pde = case["dim"], case["n"], case["pde"]
    kappa, c, b = None, None, (0.0, 0.0, 0.0)
    if pde in ("convdiff", "diffusion"):
        kappa = torch.exp(0.5 * _fourier(dim, n + 1, seed, 16 if dim == 2 else 32, 8 if dim == 2 else 6))
        if pde == "convdiff":
            b = (10.0, 0.0, 0.0)
    elif pde == "helmholtz":
        x = torch.arange(1, n + 1, device=DEV, dtype=F64) / (n + 1)
        r2 = (x[:, None] - 0.5) ** 2 + (x[None, :] - 0.5) ** 2
        c = -case["k"] ** 2 * (1.0 - 0.5 * torch.exp(-20.0 * r2))
    return {"kappa": kappa, "bvec": b, "c": c}


def _loads(case, seed, count):
    dim, n = case["dim"], case["n"]
    g = _gen(seed + 1)
    if case["pde"] == "helmholtz":  # a Gaussian source
        x0 = 0.25 + 0.5 * torch.rand(2, generator=g, device=DEV, dtype=F64)
        x = torch.arange(1, n + 1, device=DEV, dtype=F64) / (n + 1)
        r2 = (x[:, None] - x0[0]) ** 2 + (x[None, :] - x0[1]) ** 2
        return torch.exp(-r2 / (2 * 0.02 ** 2))[None]
    return torch.randn((count,) + (n,) * dim, generator=g, device=DEV, dtype=F64)


def _boundary(case, seed):
    """Smooth boundary data on the node box for the Poisson problems."""
    if case["pde"] != "poisson":
        return None
    dim, n = case["dim"], case["n"]
    a = torch.rand(dim, generator=_gen(seed + 2), device=DEV, dtype=F64)
    x = torch.arange(n + 2, device=DEV, dtype=F64) / (n + 1)
    out = torch.exp(a[0] * x).reshape((-1,) + (1,) * (dim - 1))
    for d in range(1, dim):
        out = out * torch.sin((1 + a[d]) * x).reshape([-1 if e == d else 1 for e in range(dim)])
    return out.expand((n + 2,) * dim).contiguous()


def _sensors(case, seed):
    g = _gen(seed + 3)
    N = case["n"] ** case["dim"]
    idx = torch.randperm(N, generator=g, device=DEV)[:min(256, N // 4)]
    data = 1e-3 * torch.randn(idx.numel(), generator=g, device=DEV, dtype=F64)
    return idx, data


def _options(case):
    if case["pde"] == "helmholtz":
        return ddst.SolveOptions(tol=1e-11, max_iter=3000, max_outer=20,
                                 use_hodlr=case["kind"] == "hodlr",
                                 use_hbs=case["kind"] == "sampled",
                                 basis_fp32=case["kind"] == "sampled")
    return ddst.SolveOptions(max_outer=8)


def _operator(case, coef, **kw):
    return ddst.Operator(case["dim"], case["n"], case["slabs"], precision=case["precision"],
                         **coef, **kw)


def prepare(case, seed):
    kind = case["kind"]
    coef = _problem(case, seed)
    s = {"case": case, "coef": coef, "opts": _options(case)}
    n, dim, slabs = case["n"], case["dim"], case["slabs"]
    shape = (slabs - 1, n ** (dim - 1))
    if kind in ("step", "sampled", "hodlr", "train"):
        s["f"] = _loads(case, seed, 1)[0]
        s["g"] = _boundary(case, seed)
    if kind == "solve":
        s["f"] = _loads(case, seed, case["nrhs"])
        g = _boundary(case, seed)
        s["g"] = None if g is None else g.expand((case["nrhs"],) + tuple(g.shape)).contiguous()
    if kind == "train":
        s["sensors"], s["data"] = _sensors(case, seed)
        s["kappa"] = coef["kappa"].requires_grad_()
        s["f"].requires_grad_()
    if kind in ("gmres", "apply", "compress"):
        s["x"] = torch.randn(shape, generator=_gen(seed + 4), device=DEV, dtype=F64)
        s["y"] = torch.empty(shape, device=DEV, dtype=F64)
        s["yt"] = torch.empty(shape, device=DEV, dtype=F64)
    if kind in ("solve", "hodlr", "gmres", "apply", "compress"):  # kept by the program
        s["op"] = _operator(case, coef)
    if kind == "hodlr":
        s["op"].compress(tol=1e-8, leaf=128, factor_dtype="bf16", seed=1)
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "step":
        op = _operator(case, s["coef"])
        u, gamma, _ = op.solve(s["f"], s["g"], opts=s["opts"])
        op.close()
        return u, gamma
    if kind == "solve":
        if case["nrhs"] == 1:
            return s["op"].solve(s["f"][0], None if s["g"] is None else s["g"][0], opts=s["opts"])[:2]
        return s["op"].solve_many(s["f"], s["g"], opts=s["opts"])[0]
    if kind == "train":
        u = ddst.ddst_solve(s["kappa"], s["f"], case["slabs"], bvec=s["coef"]["bvec"],
                            precision=case["precision"], opts=s["opts"])
        r = u.reshape(-1)[s["sensors"]] - s["data"]
        loss = 0.5 * (r * r).sum()
        dk, df = torch.autograd.grad(loss, (s["kappa"], s["f"]))
        return u.detach(), dk, df
    if kind == "hodlr":
        return s["op"].solve(s["f"], opts=s["opts"])[:2]
    if kind == "sampled":
        op = _operator(case, s["coef"], transfer_blocks=False)
        op.compress_hbs(rank=32, factor_dtype="bf16", seed=1)
        u, gamma, _ = op.solve(s["f"], opts=s["opts"])
        op.close()
        return u, gamma
    if kind == "compress":
        s["op"].compress(tol=1e-12, leaf=128, factor_dtype="fp64", seed=1)
        return s["op"].apply(s["x"], which="hodlr")
    if kind == "gmres":
        return s["op"].gmres(s["x"], tol=1e-8, max_iter=200)[0]
    if kind == "apply":
        s["op"].apply_noalloc(s["x"], s["y"])
        s["op"].apply_noalloc(s["x"], s["yt"], transpose=True)
        return s["y"], s["yt"]
    raise ValueError(kind)


# ---------------------------------------------------------------- work
def work(case):
    """The method's own numbers: the dense inverse of every plane's Schur
    complement of every slab (once per direction towards an interface; half
    where the operator is symmetric), the transfer chains, and the operator
    written once by a build and read once by a solve."""
    dim, n, slabs, kind = case["dim"], case["n"], case["slabs"], case["kind"]
    m, M, N, nds = (n + 1) // slabs, n ** (dim - 1), n ** dim, slabs - 1
    es = 4 if case["precision"] == "fp32" else 8
    sym = 0.5 if case["pde"] != "convdiff" else 1.0
    mat = float(M) * M
    factors, blocks, centres = slabs * (m - 1) * mat, 2.0 * (nds - 1) * mat, nds * mat
    inverses = (2 * slabs - 1) * (m - 1) + nds
    chains = 2 * (slabs - 2) * (m - 2) + 2 * (nds - 1)
    build = 2.0 * M ** 3 * (sym * inverses + chains)
    solve = 2.0 * (2 * factors + blocks + centres)  # a sweep out and back, one product
    vectors = 8.0 * 2 * N
    if kind == "step":
        return {"bytes": vectors + es * (factors + blocks + centres), "flops": build + solve}
    if kind == "solve":
        return {"bytes": vectors * case["nrhs"] + es * (factors + blocks + centres),
                "flops": solve * case["nrhs"]}
    if kind == "train":
        return {"bytes": 3 * vectors + es * (factors + blocks + centres),
                "flops": build + 2 * solve + 2.0 * M ** 3 * sym * slabs * (m - 1)}
    if kind == "hodlr":
        return {"bytes": vectors + es * (factors + centres), "flops": 2.0 * (2 * factors + centres)}
    if kind == "sampled":
        return {"bytes": vectors + es * (factors + centres),
                "flops": 2.0 * M ** 3 * sym * inverses + 2.0 * 4 * 106 * factors}
    if kind == "compress":
        return {"bytes": es * blocks, "flops": 2.0 * 2 * 32 * blocks}
    if kind == "gmres":
        return {"bytes": es * blocks, "flops": 2.0 * 18 * blocks}
    return {"bytes": 2 * es * blocks + 32.0 * nds * M, "flops": 2.0 * 2 * blocks}


# ---------------------------------------------------------------- FP64 values
class _Box:
    """The FD operator on planes lo..hi (1-based) of the grid with zero data
    around them, and its solution by restarted GMRES preconditioned with the
    constant-coefficient operator (sine transforms) scaled by sqrt(kappa)."""

    def __init__(self, case, coef, lo=1, hi=None, transpose=False):
        dim, n = case["dim"], case["n"]
        hi = n if hi is None else hi
        self.dim, self.h, nx = dim, 1.0 / (n + 1), hi - lo + 1
        self.shape = (nx,) + (n,) * (dim - 1)
        kap = coef["kappa"]
        kap = torch.ones((n + 1,) * dim, device=DEV, dtype=F64) if kap is None else kap.detach()
        self.K = []  # edge coefficients / h^2: extent + 1 along the axis
        for axis in range(dim):
            acc = 0.0
            others = [a for a in range(dim) if a != axis]
            for shifts in itertools.product((0, 1), repeat=dim - 1):
                sl = [slice(lo - 1, hi + 1) if axis == 0 else slice(None)] + [slice(None)] * (dim - 1)
                for a, sft in zip(others, shifts):
                    first = (lo - 1 if a == 0 else 0) + sft
                    sl[a] = slice(first, first + self.shape[a])
                acc = acc + kap[tuple(sl)]
            self.K.append(acc / (2 ** (dim - 1) * self.h ** 2))
        sign = -1.0 if transpose else 1.0
        self.b = [sign * v / (2 * self.h) for v in coef["bvec"][:dim]]
        self.c = None if coef["c"] is None else coef["c"][lo - 1:hi]
        diag = sum(self._side(a, 0) + self._side(a, 1) for a in range(dim)) / (2 * dim / self.h ** 2)
        self.scale = 1.0 / torch.sqrt(diag)
        shift = 0.0 if self.c is None else float(self.c.mean())
        self.Q, lam = [], torch.full(self.shape, shift, device=DEV, dtype=F64)
        for a, ext in enumerate(self.shape):
            i = torch.arange(1, ext + 1, device=DEV, dtype=F64)
            self.Q.append(math.sqrt(2 / (ext + 1)) * torch.sin(math.pi * (i[:, None] * i[None, :]) / (ext + 1)))
            e = 4 / self.h ** 2 * torch.sin(math.pi * i / (2 * (ext + 1))) ** 2
            lam = lam + e.reshape([-1 if a == d else 1 for d in range(dim)])
        self.lam = lam

    def _side(self, axis, up):
        return self.K[axis].narrow(axis, up, self.shape[axis])

    def apply(self, box):
        """A u on the box; `box` has one more layer of nodes on each side."""
        inner = tuple(slice(1, -1) for _ in range(self.dim))
        u = box[inner]
        out = torch.zeros_like(u) if self.c is None else self.c * u
        for a in range(self.dim):
            sl = list(inner)
            sl[a] = slice(2, None)
            up = box[tuple(sl)]
            sl[a] = slice(0, -2)
            dn = box[tuple(sl)]
            out = out + self._side(a, 1) * (u - up) + self._side(a, 0) * (u - dn) + self.b[a] * (up - dn)
        return out

    def pad(self, u):
        return torch.nn.functional.pad(u, (1, 1) * self.dim)

    def _sine(self, v):
        for a, q in enumerate(self.Q):
            v = torch.tensordot(q, v.movedim(a, 0), dims=1).movedim(0, a)
        return v

    def precondition(self, r):
        return self.scale * self._sine(self._sine(self.scale * r) / self.lam)

    def solve(self, b, restart=400, cycles=12):
        u = torch.zeros_like(b)
        bn = float(b.norm())
        N = b.numel()
        if bn == 0.0:
            return u
        last = math.inf
        for _ in range(cycles):
            r = b - self.apply(self.pad(u))
            beta = float(r.norm())
            if beta <= 1e-16 * bn or beta > 0.5 * last:  # no longer improving
                break
            last = beta
            V = [r.reshape(-1) / beta]
            H = torch.zeros(restart + 1, restart, dtype=F64)
            basis = torch.empty(min(restart, 32) + 1, N, device=DEV, dtype=F64)
            basis[0] = V[0]
            y, k = None, 0
            for k in range(restart):
                if k + 2 > basis.shape[0]:
                    basis = torch.cat([basis, torch.empty(min(basis.shape[0], 200), N, device=DEV, dtype=F64)])
                z = self.precondition(basis[k].reshape(self.shape))
                w = self.apply(self.pad(z)).reshape(-1)
                hcol = torch.zeros(k + 1, device=DEV, dtype=F64)
                for _again in range(2):
                    d = basis[:k + 1] @ w
                    w = w - basis[:k + 1].T @ d
                    hcol += d
                nw = float(w.norm())
                H[:k + 1, k] = hcol.cpu()
                H[k + 1, k] = nw
                basis[k + 1] = w / nw
                if k % 10 == 9 or k + 1 == restart:
                    e = torch.zeros(k + 2, 1, dtype=F64)
                    e[0] = beta
                    y = torch.linalg.lstsq(H[:k + 2, :k + 1], e).solution
                    if float((H[:k + 2, :k + 1] @ y - e).norm()) <= 1e-11 * beta:
                        break
            u = u + self.precondition((basis[:k + 1].T @ y.to(DEV)).reshape(self.shape))
        res = float((b - self.apply(self.pad(u))).norm())
        if not res <= 1e-8 * bn:
            raise RuntimeError("reference solve: relative residual %.2g" % (res / bn))
        return u


def _global(case, coef, f, g):
    """Solution and interface traces of A u = f, u = g on the boundary."""
    box = _Box(case, coef)
    rhs = f
    if g is not None:
        ring = g.clone()
        ring[tuple(slice(1, -1) for _ in range(case["dim"]))] = 0.0
        rhs = f - box.apply(ring)
    u = box.solve(rhs)
    m = (case["n"] + 1) // case["slabs"]
    return u, u[m - 1::m].reshape(case["slabs"] - 1, -1)


def _product(case, coef, x, transpose):
    """S x (or S^T x): row j of S is the centre trace of the double slab's
    solution for traces on its two sides; S^T by the transposed local solves."""
    n, dim, slabs = case["n"], case["dim"], case["slabs"]
    m, nds = (n + 1) // slabs, slabs - 1
    plane = (n,) * (dim - 1)
    x = x.reshape((nds,) + plane)
    y = x.clone()
    for j in range(1, nds + 1):
        lo, hi = (j - 1) * m + 1, (j + 1) * m - 1
        box = _Box(case, coef, lo, hi)
        if not transpose:
            ring = torch.zeros([e + 2 for e in box.shape], device=DEV, dtype=F64)
            inner = (slice(1, -1),) * (dim - 1)
            if j >= 2:
                ring[(0,) + inner] = x[j - 2]
            if j < nds:
                ring[(-1,) + inner] = x[j]
            y[j - 1] -= box.solve(-box.apply(ring))[m - 1]
        else:
            adj = _Box(case, coef, lo, hi, transpose=True)
            r = torch.zeros(box.shape, device=DEV, dtype=F64)
            r[m - 1] = x[j - 1]
            z = adj.solve(r)  # A^{-T} R^T x_j; S_{j,j'}^T x_j = -A(I,J)^T z
            if j >= 2:
                y[j - 2] += (-box._side(0, 0)[0] - box.b[0]) * z[0]
            if j < nds:
                y[j] += (-box._side(0, 1)[-1] + box.b[0]) * z[-1]
    return y.reshape(nds, -1)


def _poisson_interface(case, x):
    """S^{-1} x for the Poisson operator by separation of variables: the
    eigenvalues are 1 - cos(r pi / N_s) / T_m(1 + lambda_q h^2 / 2)."""
    n, dim, slabs = case["n"], case["dim"], case["slabs"]
    m, nds = (n + 1) // slabs, slabs - 1

    def sine(ext):
        i = torch.arange(1, ext + 1, device=DEV, dtype=F64)
        return math.sqrt(2 / (ext + 1)) * torch.sin(math.pi * (i[:, None] * i[None, :]) / (ext + 1))

    i = torch.arange(1, n + 1, device=DEV, dtype=F64)
    e = 4 * torch.sin(math.pi * i / (2 * (n + 1))) ** 2
    lam = e if dim == 2 else e[:, None] + e[None, :]
    s = 1.0 / torch.cosh(m * torch.acosh(1 + lam / 2))
    r = torch.arange(1, nds + 1, device=DEV, dtype=F64)
    ev = 1 - s[None] * torch.cos(math.pi * r / slabs).reshape((-1,) + (1,) * (dim - 1))
    qs = [sine(nds)] + [sine(n)] * (dim - 1)

    def transform(v):
        for a, q in enumerate(qs):
            v = torch.tensordot(q, v.movedim(a, 0), dims=1).movedim(0, a)
        return v

    v = x.reshape((nds,) + (n,) * (dim - 1))
    return transform(transform(v) / ev).reshape(nds, -1)


def _cell_gradient(case, u, lam):
    dim, n = case["dim"], case["n"]
    U, L = torch.nn.functional.pad(u, (1, 1) * dim), torch.nn.functional.pad(lam, (1, 1) * dim)
    out = torch.zeros((n + 1,) * dim, device=DEV, dtype=F64)
    for axis in range(dim):
        for shifts in itertools.product((0, 1), repeat=dim - 1):
            lo = [slice(0, n + 1)] * dim
            for a, sft in zip([a for a in range(dim) if a != axis], shifts):
                lo[a] = slice(sft, sft + n + 1)
            hi = list(lo)
            hi[axis] = slice(1, n + 2)
            out += (L[tuple(lo)] - L[tuple(hi)]) * (U[tuple(lo)] - U[tuple(hi)])
    return -out * (n + 1) ** 2 / 2 ** (dim - 1)


def exact(case, seed):
    kind = case["kind"]
    coef = _problem(case, seed)
    shape = (case["slabs"] - 1, case["n"] ** (case["dim"] - 1))
    if kind in ("step", "hodlr", "sampled"):
        return _global(case, coef, _loads(case, seed, 1)[0], _boundary(case, seed))
    if kind == "solve":
        g = _boundary(case, seed)
        F = _loads(case, seed, case["nrhs"])
        if case["nrhs"] == 1:
            return _global(case, coef, F[0], g)
        return torch.stack([_global(case, coef, f, g)[0] for f in F])
    if kind == "train":
        u, _ = _global(case, coef, _loads(case, seed, 1)[0], None)
        idx, data = _sensors(case, seed)
        gbar = torch.zeros(u.numel(), device=DEV, dtype=F64)
        gbar[idx] = u.reshape(-1)[idx] - data
        lam = _Box(case, coef, transpose=True).solve(gbar.reshape(u.shape))
        return u, _cell_gradient(case, u, lam), lam
    x = torch.randn(shape, generator=_gen(seed + 4), device=DEV, dtype=F64)
    if kind == "gmres":
        return _poisson_interface(case, x)
    if kind == "compress":
        return _product(case, coef, x, False)
    return _product(case, coef, x, False), _product(case, coef, x, True)
