"""Performance cases: the calls a program around this library makes, timed through its
public Python entry points.

The meshes are boxes in LDU form, as in meshgen/boxes.py: a finite-volume hex mesh graded
towards a wall ("graded", aspect ratio up to 100), and boxes with lognormal coefficients
("lognormal").  Cells are numbered as a mesh generator leaves them ("natural"), by level
sets from a corner, which is what a Cuthill-McKee renumbering gives on a box ("levels"), or
at random ("shuffled").  Inputs are built on the GPU from a seed, and right-hand sides are
A x for a known x, so that exact() can state the solution.
"""
from __future__ import annotations

import math

import torch

from paper_2512_22215_amd import LduMatrix, ldu_solve

# The two hierarchies the benchmark runs: pairwise matching on every level, and three
# matching passes per level below the first.  One Jacobi sweep before and after the
# coarse correction: the setting of CG with a V-cycle.
PAIRWISE = {"n_pre": 1, "n_post": 1}
MERGED = {"n_pre": 1, "n_post": 1, "passes": 3, "aggressive_from": 1}


def _case(name, do, nx, ny, nz, coeff="lognormal", order="natural", **kw):
    return dict(name=name, do=do, nx=nx, ny=ny, nz=nz, coeff=coeff, order=order, **kw)


def listed():
    return [
        # one product with the 8M-cell graded matrix: the kernel that every solver runs
        _case("amul_200", "amul", 200, 200, 200, "graded", dtype="f64", transposed=False),
        # one FP32 product on a small renumbered mesh: a call bound by its launch
        _case("amul_f32_small", "amul", 48, 40, 36, order="levels", dtype="f32",
              transposed=False),
        # diagonal CG on a small mesh: about a hundred short iterations
        _case("pcg_32", "pcg", 32, 32, 32, precision="fp64"),
        # diagonal CG on the million-cell box
        _case("pcg_100", "pcg", 100, 100, 100, precision="fp64"),
        # CG with a V-cycle on the million-cell box, the default pairwise hierarchy
        _case("pcg_gamg_100", "pcg_gamg", 100, 100, 100, precision="fp64", merged=False),
        # the 8M-cell graded pressure solve of the benchmark
        _case("pcg_gamg_200", "pcg_gamg", 200, 200, 200, "graded", precision="fp64",
              merged=True),
        # FP32 CG and V-cycle inside FP64 refinement, to full accuracy
        _case("mixed_128", "pcg_gamg", 128, 128, 128, order="levels", precision="mixed",
              merged=True),
        # GAMG as a solver, default settings, on a mesh that was never renumbered
        _case("gamg_128", "gamg", 128, 128, 128, order="shuffled", precision="fp64"),
        # one pressure step of a SIMPLE loop: assembly from geometry, the hierarchy's
        # values, and a loose solve for the pressure correction
        _case("step_151", "step", 151, 143, 139, "graded", merged=True),
        # differentiable solve: forward, adjoint and the coefficient gradients
        _case("autograd_100", "autograd", 100, 100, 100, precision="fp64"),
        # PBiCG on the convection-diffusion box (an implicit velocity equation)
        _case("pbicg_100", "pbicg", 100, 100, 100, "upwind"),
        # a new mesh: matrix, hierarchy and first solve
        _case("cold_121", "cold", 121, 117, 130, order="levels", merged=True),
    ]


# cells that a drawn case of each kind spans
RANGE = {"amul": (4e3, 8e6), "pcg": (4e3, 1e6), "pcg_gamg": (4e3, 4e6), "gamg": (4e3, 2e6),
         "step": (3e4, 3e6), "autograd": (4e3, 1e6), "pbicg": (4e3, 2e6), "cold": (2e4, 2e6)}


def draw(rng):
    do = rng.choice(sorted(RANGE))
    lo, hi = RANGE[do]
    side = math.exp(rng.uniform(math.log(lo), math.log(hi))) ** (1 / 3)
    # box proportions within about 1 : 1.6, the product within the range
    a, b = rng.uniform(0.8, 1.25), rng.uniform(0.8, 1.25)
    nx, ny, nz = (max(8, int(side * f)) for f in (a, b, 0.98 / (a * b)))
    order = rng.choice(["natural", "natural", "levels", "levels", "shuffled"])
    coeff = {"step": "graded", "pbicg": "upwind"}.get(do) or (
        rng.choice(["lognormal", "lognormal", "graded"]) if do in ("amul", "pcg_gamg")
        else "lognormal")
    c = dict(do=do, nx=nx, ny=ny, nz=nz, coeff=coeff, order=order)
    if do == "amul":
        c["dtype"] = rng.choice(["f64", "f64", "f32"])
        c["transposed"] = c["dtype"] == "f64" and rng.random() < 0.4
    if do in ("pcg", "pcg_gamg", "gamg", "autograd"):
        c["precision"] = "fp64" if coeff == "graded" else rng.choice(["fp64", "fp64", "mixed"])
    if do in ("pcg_gamg", "step", "cold"):
        c["merged"] = rng.random() < 0.5
    return c


# ------------------------------------------------------------------------ meshes
class Box:
    """A box matrix in structured form: diag[N], up[N, 3] = A[i, i + stride_k] and
    low[N, 3] = A[i + stride_k, i] (0 where cell i has no neighbour along axis k)."""

    def __init__(self, case, seed):
        self.shape = nx, ny, nz = case["nx"], case["ny"], case["nz"]
        self.n = n = nx * ny * nz
        self.strides = (1, nx, nx * ny)
        self.gen = torch.Generator(device="cuda").manual_seed(1000 * seed + 17)
        i = torch.arange(n, device="cuda")
        self.pos = pos = torch.stack([i % nx, (i // nx) % ny, i // (nx * ny)], 1)
        self.mask = pos < torch.tensor([nx - 1, ny - 1, nz - 1], device="cuda")
        {"graded": self._graded, "lognormal": self._lognormal,
         "upwind": self._upwind}[case["coeff"]]()
        self._number(case["order"])

    def randn(self, *size):
        return torch.randn(*size, generator=self.gen, device="cuda", dtype=torch.float64)

    def spacing(self):
        nz = self.shape[2]
        dx = 1.0 / nz
        k = torch.arange(nz, device="cuda", dtype=torch.float64)
        return dx, torch.clamp(dx / 100.0 * 1.05 ** k, max=dx)

    def _symmetric(self, a, boundary):
        a = a * self.mask
        d = a.sum(1)
        for k, s in enumerate(self.strides):
            d[s:] += a[:-s, k]
        self.up = self.low = a
        self.diag = -(d + boundary)

    def _lognormal(self):
        a = torch.exp(0.5 * self.randn(self.n, 3))
        self._symmetric(a, 2.0 * (self.pos[:, 0] == 0))  # Dirichlet at x = 0

    def _graded(self):
        dx, dz = self.spacing()
        kz = self.pos[:, 2]
        dz0, dz1 = dz[kz], dz[torch.clamp(kz + 1, max=self.shape[2] - 1)]
        a = torch.stack([dz0, dz0, dx * dx / (0.5 * (dz0 + dz1))], 1)
        u = torch.rand(self.n, 3, generator=self.gen, device="cuda", dtype=torch.float64)
        top = kz == self.shape[2] - 1  # Dirichlet at the top layer
        self._symmetric(a * (0.95 + 0.1 * u), top * (dx * dx / (0.5 * dz[-1])))

    def _upwind(self):
        h = 1.0 / self.shape[0]
        vel = torch.tensor([1.0, 0.5, 0.25], device="cuda", dtype=torch.float64)
        nu = torch.exp(0.5 * self.randn(self.n, 3)) * h
        diff = nu * h * self.mask
        flux = vel * h * h * self.mask
        self.up, self.low = -diff, -(diff + flux)
        # one implicit Euler step at Courant number 2; outflow at the far faces
        d = torch.full((self.n,), h ** 3 / (2.0 * h / float(vel.norm())), device="cuda",
                       dtype=torch.float64)
        d += (diff + flux).sum(1) + (vel * h * h * ~self.mask).sum(1)
        for k, s in enumerate(self.strides):
            d[s:] += diff[:-s, k]
        self.diag = d + 2.0 * h * h * (self.pos[:, 0] == 0)

    def _number(self, order):
        if order == "natural":
            self.new = None
        elif order == "levels":
            at = torch.sort(self.pos.sum(1), stable=True).indices
            self.new = torch.empty_like(at)
            self.new[at] = torch.arange(self.n, device="cuda")
        else:
            self.new = torch.randperm(self.n, generator=self.gen, device="cuda")

    def product(self, x, transposed=False):
        up, low = (self.low, self.up) if transposed else (self.up, self.low)
        y = self.diag * x
        for k, s in enumerate(self.strides):
            y[:-s] += up[:-s, k] * x[s:]
            y[s:] += low[:-s, k] * x[:-s]
        return y

    def field(self, noise=0.01):
        """A pressure-like field: a few long waves and some noise."""
        p = self.pos.to(torch.float64) + 0.5
        x = noise * self.randn(self.n)
        w = self.randn(4, 4)
        for k in range(4):
            f = torch.ones_like(x)
            for j, m in enumerate(self.shape):
                f = f * torch.cos(math.pi * (1 + (k + j) % 3) * p[:, j] / m + w[k, j])
            x = x + w[k, 3] * f
        return x

    def cells(self, v):
        """A cell field in the mesh's numbering."""
        if self.new is None:
            return v.contiguous()
        out = torch.empty_like(v)
        out[self.new] = v
        return out

    def faces(self):
        """owner, neighbour (sorted) and f(v_up, v_low): face fields for the owner-to-
        neighbour and the neighbour-to-owner direction."""
        flat = torch.nonzero(self.mask.reshape(-1)).squeeze(1)
        own = flat // 3
        nb = own + torch.tensor(self.strides, device="cuda")[flat % 3]
        if self.new is None:
            return own.int(), nb.int(), lambda u, l: (u.reshape(-1)[flat], l.reshape(-1)[flat])
        o, b = self.new[own], self.new[nb]
        flip = o > b
        lo, hi = torch.minimum(o, b), torch.maximum(o, b)
        at = torch.sort(lo * self.n + hi).indices

        def pick(u, l):
            u, l = u.reshape(-1)[flat], l.reshape(-1)[flat]
            return torch.where(flip, l, u)[at], torch.where(flip, u, l)[at]
        return lo[at].int(), hi[at].int(), pick

    def arrays(self):
        own, nb, pick = self.faces()
        up, low = pick(self.up, self.low)
        return self.n, own, nb, self.cells(self.diag), up, low


# ------------------------------------------------------------------------ cases
def _opts(case):
    """Solver options: 1e-8 as in the benchmark; refinement and gradients go to full
    accuracy."""
    do, o = case["do"], {}
    if do in ("pcg", "pcg_gamg", "gamg", "autograd"):
        o["precision"] = case["precision"]
    o["rel_tol"] = 1e-11 if do == "autograd" or case.get("precision") == "mixed" else 1e-8
    if do == "step":
        o["rel_tol"] = 1e-2
    if do == "pbicg":
        o["rel_tol"] = 1e-11
    if do in ("pcg_gamg", "autograd", "step", "cold"):
        o["precond"] = 2
    return o


def _hierarchy(case):
    return dict(MERGED if case.get("merged") else PAIRWISE)


def prepare(case, seed):
    box = Box(case, seed)
    do = case["do"]
    s = {"do": do, "opts": _opts(case), "dtype": case.get("dtype"),
         "transposed": case.get("transposed", False), "hierarchy": _hierarchy(case)}
    n, own, nb, diag, up, low = box.arrays()
    x = box.field()
    if do == "cold":
        s["arrays"] = (n, own, nb, diag, up, low)
        s["b"] = box.cells(box.product(x))
        return s
    m = s["m"] = LduMatrix(n, own, nb, diag, up, low)
    if do == "amul":
        s["x"] = box.cells(x).to(torch.float32 if case["dtype"] == "f32" else torch.float64)
        s["y"] = torch.empty_like(s["x"])
        return s
    s["b"] = box.cells(box.product(x))
    if do in ("pcg_gamg", "autograd", "step"):
        m.gamg_setup(**s["hierarchy"])
    elif do == "gamg":
        m.gamg_setup()
    if do == "autograd":
        s["leaves"] = [t.requires_grad_() for t in (diag, up, low, s["b"])]
        s["gx"] = box.cells(box.product(box.field(), True))
    if do == "step":
        s["geometry"] = _geometry(box)
    return s


def _geometry(box):
    """Arguments of assemble_pressure on the graded box: 1/A_p as a lognormal field, a
    random face flux, a Dirichlet top layer."""
    dx, dz = box.spacing()
    kz = box.pos[:, 2]
    dz0, dz1 = dz[kz], dz[torch.clamp(kz + 1, max=box.shape[2] - 1)]
    area = torch.stack([dx * dz0, dx * dz0, torch.full_like(dz0, dx * dx)], 1)
    delta = torch.stack([torch.full_like(dz0, 1 / dx)] * 2 + [1 / (0.5 * (dz0 + dz1))], 1)
    w = torch.stack([torch.full_like(dz0, 0.5)] * 2 + [dz1 / (dz0 + dz1)], 1)
    gamma = torch.exp(0.3 * box.randn(box.n))
    top = kz == box.shape[2] - 1
    diag_bc = torch.where(top, gamma * dx * dx / (0.5 * dz[-1]), torch.zeros_like(gamma))
    phi = box.randn(box.n, 3) * dx * dx
    _, _, pick = box.faces()
    face = lambda u, l: pick(u, l)[0].contiguous()  # noqa: E731
    return {"gamma": box.cells(gamma), "weights": face(w, 1.0 - w),
            "mag_sf": face(area, area), "delta": face(delta, delta),
            "diag_bc": box.cells(diag_bc), "phi": face(phi, -phi)}


def run(s):
    do, m, o = s["do"], s.get("m"), s["opts"]
    if do == "amul":
        f = m.amul_f32 if s["dtype"] == "f32" else m.tmul if s["transposed"] else m.amul
        return f(s["x"], out=s["y"])
    if do in ("pcg", "pcg_gamg"):
        return m.pcg(s["b"], **o)[0]
    if do == "gamg":
        return m.gamg(s["b"], **o)[0]
    if do == "pbicg":
        return m.pbicg(s["b"], **o)[0]
    if do == "step":
        b = m.assemble_pressure(**s["geometry"])
        return {"b": b, "x": m.pcg(b, **o)[0]}
    if do == "autograd":
        x = ldu_solve(*s["leaves"], m, method="pcg", **o)
        return [x.detach(), *torch.autograd.grad(x, s["leaves"], s["gx"])]
    m = LduMatrix(*s["arrays"])  # cold
    m.gamg_setup(**s["hierarchy"])
    x = m.pcg(s["b"], **o)[0]
    m.close()
    return x


def exact(case, seed):
    box = Box(case, seed)
    x = box.field()
    do = case["do"]
    if do == "amul":
        if case["dtype"] == "f32":
            x = x.to(torch.float32).to(torch.float64)
        return box.cells(box.product(x, case["transposed"]))
    if do == "autograd":
        lam = box.field()
        up, low = -lam[:, None] * _at(box, x), -_at(box, lam) * x[:, None]
        gu, gl = box.faces()[2](up, low)
        return [box.cells(x), box.cells(-lam * x), gu, gl, box.cells(lam)]
    if do == "step":  # a loose solve has no value of its own
        g = _geometry(box)
        own, nb, _ = box.faces()
        b = torch.zeros(box.n, device="cuda", dtype=torch.float64)
        b.index_add_(0, own.long(), g["phi"])
        b.index_add_(0, nb.long(), -g["phi"])
        return {"b": b, "x": None}
    return box.cells(x)


def _at(box, v):
    """v at the neighbour along each axis."""
    out = torch.zeros(box.n, 3, device="cuda", dtype=torch.float64)
    for k, s in enumerate(box.strides):
        out[:-s, k] = v[s:]
    return out


def work(case):
    """Bytes and operations of one pass: a product reads the LDU arrays (24 bytes per cell
    and per face in FP64, 12 and 16 in FP32) and a solve makes its iterations' products.
    The iteration counts are typical ones: they grow with the box's side for diagonal CG,
    slowly for the multigrid forms."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    n = nx * ny * nz
    f = 3 * n - nx * ny - ny * nz - nx * nz
    do = case["do"]
    prod, vec = 24 * n + 24 * f, 8 * n
    flops = 2 * (n + 2 * f)
    if do == "amul":
        return {"bytes": 12 * n + 16 * f if case["dtype"] == "f32" else prod, "flops": flops}
    side = n ** (1 / 3)
    if do == "pcg":  # product, r update, direction and x update
        it = 7.0 * side * (1.25 if case["precision"] == "mixed" else 1.0)
        return {"bytes": it * (prod + 10 * vec), "flops": it * (flops + 12 * n)}
    if do == "pbicg":
        it = 0.6 * side + 10
        return {"bytes": it * (prod + 16 * f + 16 * vec), "flops": it * (2 * flops + 20 * n)}
    # a V-cycle with one sweep each side passes over level 0 twice; the coarse levels
    # together hold about as much again
    cycle = 2 * (2 * prod) + 6 * vec
    if do == "gamg":
        it = 25
        return {"bytes": it * (2 * cycle + prod), "flops": it * 11 * flops}
    it = (0.75 if case["coeff"] == "graded" else 0.55) * side
    it *= {"autograd": 2.6, "step": 0.1}.get(do, 1.0)
    it *= 1.5 if case.get("precision") == "mixed" else 1.0
    it += 1
    more = {"step": 4 * prod, "cold": 10 * prod, "autograd": 6 * prod}.get(do, 0)
    half = 0.6 if case.get("precision") == "mixed" else 1.0
    return {"bytes": half * it * (cycle + prod + 8 * vec) + more, "flops": it * 6 * flops}
