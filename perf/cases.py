"""Workloads that the framework's performance is measured on.

Each case is one pass through the public entry points as a simulation calls
them: an operator application inside somebody's own Krylov or time loop, a
whole solve, a differentiable heat step, or the interface terms of a time
step.  Meshes, material data, level sets and tolerances are those of
``workloads.py``, the benchmark and the tests; the ragged sizes are meshes
whose edges are no multiples of a brick.  Fields vary with the seed: the
place and size of the liquid region, the melt temperature, the vectors.

``exact`` evaluates the same results in plain float64 torch: dense 27 x 27
cell tables in place of sum factorization, and for a solve the solution that
its right-hand side was made from, or a conjugate gradient iteration taken
down to rounding.
"""
import math

import torch

from paper_2501_18781_amd import autograd, mf, picard
from paper_2501_18781_amd import workloads as W

DEV = "cuda"
F64 = torch.float64

# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------


def _case(kind, n, **kw):
    c = {"kind": kind, "nx": n[0], "ny": n[1], "nz": n[2], "walls": W.ALL_FACES, "equal_edges": True,
         "form": "linear", "transpose": False, "dt": 1.0e-4 if "oseen" in kind else 1.0e-3}
    if kind == "heat":
        c["dtype"], c["coefficients"] = "float64", "levelset"
    c.update(kw)
    return c


def listed():
    cases = [
        # the smoke and test mesh: two launches on eight bricks, latency counts
        dict(_case("heat", (8, 8, 8), walls=0), name="heat_8"),
        # the benchmark's operator application
        dict(_case("heat", (64, 64, 64)), name="heat_64"),
        # the paper's sine Heaviside, unequal cell edges, clipped bricks, mixed walls
        dict(_case("heat", (50, 37, 61), form="sine", equal_edges=False, walls=W.FACE_ZLO | W.FACE_XHI),
             name="heat_sine_50x37x61"),
        # a finest multigrid level in single precision
        dict(_case("heat", (128, 128, 128), dtype="float32"), name="heat_fp32_128"),
        # convection, adjoint direction (adjoint solves), ragged
        dict(_case("heat_conv", (45, 64, 51), transpose=True), name="heat_conv_transposed_45x64x51"),
        # the benchmark's momentum operator
        dict(_case("oseen", (48, 48, 48)), name="oseen_48"),
        # momentum across the melting range (Darcy damping), sine Heaviside, adjoint direction
        dict(_case("oseen_melt", (33, 41, 29), form="sine", transpose=True, equal_edges=False),
             name="oseen_melt_transposed_33x41x29"),
        # the benchmark's Jacobi-CG solve of one implicit heat step
        dict(_case("cg", (64, 64, 64), rtol=1e-10), name="cg_64"),
        # the benchmark's momentum solve
        dict(_case("gmres_oseen", (48, 48, 48), rtol=1e-8), name="gmres_oseen_48"),
        # multigrid-preconditioned heat solve where mass and conduction are comparable
        dict(_case("mg", (128, 128, 128), dt=1.0, rtol=1e-8, coarse=4), name="mg_128"),
        # one differentiable heat step, forward and backward (gradient-based fitting)
        dict(_case("step", (32, 32, 32), form="sine"), name="heat_step_gradient_32"),
        # once per time step: interface heat sources and the level-set transport velocity
        dict(_case("interface", (64, 64, 64), form="sine"), name="interface_terms_64"),
    ]
    return cases


# kind, share of the draws, edge of the smallest and of the largest cube
_RANGES = [("heat", 4, 8, 112), ("heat_conv", 2, 8, 80), ("heat_melt", 1, 8, 80), ("oseen", 3, 8, 56),
           ("oseen_melt", 1, 8, 48), ("cg", 2, 8, 80), ("gmres_oseen", 2, 8, 40), ("gmres_conv", 1, 8, 56),
           ("mg", 1, 16, 112), ("step", 2, 8, 48), ("picard", 1, 8, 48), ("interface", 2, 8, 80)]


def draw(rng):
    kind, _, lo, hi = rng.choices(_RANGES, weights=[r[1] for r in _RANGES])[0]
    edge = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    if kind == "mg":
        # every direction halves down to the coarse mesh
        halvings = max(1, round(math.log2(edge / rng.choice([3, 4, 5]))))
        coarse = [max(2, round(edge / 2 ** halvings * 2 ** rng.uniform(-0.2, 0.2))) for _ in range(3)]
        n = [c << halvings for c in coarse]
    else:
        n = [max(4, round(edge * 2 ** rng.uniform(-0.35, 0.25))) for _ in range(3)]
    if rng.random() < 0.2 and kind != "mg":
        n = [max(4, round(edge / 4) * 4)] * 3
    c = _case(kind, n, form=rng.choice(["linear", "sine"]), equal_edges=rng.random() < 0.6,
              walls=rng.choice([W.ALL_FACES, W.ALL_FACES, 0, rng.randrange(64)]))
    if kind in ("heat", "heat_conv", "heat_melt", "oseen", "oseen_melt"):
        c["transpose"] = kind != "heat" and rng.random() < 0.4
    if kind == "heat":
        c["dtype"] = rng.choice(["float64", "float64", "float32"])
        c["coefficients"] = rng.choice(["levelset", "levelset", "levelset", "points"])
    if kind == "cg":
        c["rtol"], c["dt"] = 1e-10, rng.choice([1e-3, 1e-3, 1.0])
    if kind in ("gmres_oseen", "gmres_conv"):
        c["rtol"] = 1e-8
    if kind == "mg":
        c["rtol"], c["dt"], c["coarse"] = 1e-8, rng.choice([1e-3, 1.0, 1e3]), coarse[0]
    if kind == "picard":
        c["dt"] = rng.choice([1e-3, 1.0])
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

class Inputs:
    """The seeded fields of a case, float64 on the GPU in node order (x fastest)."""

    def __init__(self, case, seed):
        g = torch.Generator(device="cpu").manual_seed(1000003 * seed + 7)
        r = torch.rand(24, generator=g, dtype=F64).tolist()
        n = (case["nx"], case["ny"], case["nz"])
        hi = tuple(c / max(n) for c in n) if case["equal_edges"] else (1.0, 1.0, 1.0)
        self.mesh = W.Mesh(n, hi=hi, dirichlet=case["walls"])
        self.N = tuple(2 * c + 1 for c in n)
        self.nn = self.N[0] * self.N[1] * self.N[2]
        eps = 2.0 * max(self.mesh.h)
        hkind = 1 if case["form"] == "sine" else 0
        self.eps = eps
        melt = "melt" in case["kind"] or case["kind"] == "picard"
        self.heat = W.HeatParams(dt=case["dt"], heaviside=hkind, eps=eps, penalty=2.0e9 if melt else 0.0)
        self.flow = W.OseenParams(dt=case["dt"], heaviside=hkind, eps=eps)
        x, y, z = self.axes = [torch.linspace(0.0, hi[d], self.N[d], dtype=F64, device=DEV) for d in range(3)]
        X, Y, Z = x[None, None, :], y[None, :, None], z[:, None, None]
        self.X, self.Y, self.Z, self.hi = X, Y, Z, hi
        if "oseen" in case["kind"]:
            zs = hi[2] * (0.45 + 0.1 * r[0]) + 0.05 * hi[2] * torch.cos(2 * math.pi * X) * torch.cos(2 * math.pi * Y)
            d = zs - Z
        else:
            c = [hi[k] * (0.42 + 0.16 * r[k]) for k in range(3)]
            d = (0.26 + 0.08 * r[3]) * min(hi) - torch.sqrt((X - c[0]) ** 2 + (Y - c[1]) ** 2 + (Z - c[2]) ** 2)
        self.phi = self.flat(torch.tanh(d / (2.0 * eps)))
        self.r = r
        self.gen = torch.Generator(device=DEV).manual_seed(seed)

    def flat(self, f):
        return f.expand(self.N[2], self.N[1], self.N[0]).contiguous().reshape(-1)

    def uniform(self, comps=1):
        return torch.rand(comps * self.nn, generator=self.gen, dtype=F64, device=DEV) * 2.0 - 1.0

    def smooth(self):
        """A temperature-like field that vanishes on the walls of the box."""
        t = 0.0
        for k in range(3):
            a = 1.0 if k == 0 else 0.3 * (self.r[4 + k] - 0.5)
            t = t + a * (torch.sin(math.pi * (1 + k) * self.X / self.hi[0]) * torch.sin(math.pi * self.Y / self.hi[1]) *
                         torch.sin(math.pi * (1 + k) * self.Z / self.hi[2]))
        return self.flat(t)

    def velocity(self):
        s = 0.6 + 0.8 * self.r[8]
        px, py, pz = math.pi * self.X, math.pi * self.Y, math.pi * self.Z
        u = self.flat(s * torch.sin(px) * torch.cos(py) * torch.cos(pz))
        v = self.flat(-s * torch.cos(px) * torch.sin(py) * torch.cos(pz))
        w = self.flat(0.1 * s * torch.sin(px) * torch.sin(py) * torch.sin(pz))
        return torch.cat([u, v, w])

    def melt_temperature(self):
        t = 1800.0 + 600.0 * self.Z / self.hi[2] + 40.0 * (self.r[9] - 0.5) * torch.cos(2 * math.pi * self.X)
        return self.flat(t + 0.0 * self.Y)

    def boiling_temperature(self, boil):
        t = 300.0 * (self.Z - 0.5) + 100.0 * self.r[10] * torch.cos(2 * math.pi * self.X) * torch.cos(2 * math.pi * self.Y)
        return self.flat(boil + t)

    def point_coefficients(self, cells):
        H = torch.rand(cells * 27, generator=self.gen, dtype=F64, device=DEV)
        p = self.heat
        return p.k_g + H * (p.k_l - p.k_g), p.rc_g + H * (p.rc_l - p.rc_g)


def _fields(case, seed):
    """(inputs, dict of the tensors a case works on)."""
    q = Inputs(case, seed)
    kind = case["kind"]
    f = {"phi": q.phi}
    if kind in ("heat", "heat_conv", "heat_melt"):
        f["x"] = q.uniform()
    if kind in ("oseen", "oseen_melt", "gmres_oseen"):
        f["x"] = q.uniform(3)
    if kind == "gmres_conv":
        f["x"] = q.uniform()
    if kind in ("cg", "mg", "step"):
        f["x"] = q.smooth()
    if kind in ("heat_conv", "gmres_conv", "oseen", "oseen_melt", "gmres_oseen", "interface"):
        f["u0"] = q.velocity()
    if kind in ("heat_melt", "oseen_melt", "picard"):
        f["Tc"] = q.melt_temperature()
    if kind == "interface":
        f["T"] = q.boiling_temperature(W.SourceParams().T_boil)
    if kind == "heat" and case["coefficients"] == "points":
        f["kq"], f["rcq"] = q.point_coefficients(q.mesh.n_cells)
    if kind == "heat" and case["dtype"] == "float32":
        f = {k: v.float() for k, v in f.items()}
    return q, f


def prepare(case, seed):
    q, f = _fields(case, seed)
    kind = case["kind"]
    ctx = mf.Context(q.mesh)
    s = {"kind": kind, "ctx": ctx, "case": case}
    if kind == "heat":
        prec = mf.MF_FP32 if case["dtype"] == "float32" else mf.MF_FP64
        if case["coefficients"] == "points":
            s["op"] = mf.heat_operator(ctx, q.heat, k_q=f["kq"], rc_q=f["rcq"], precision=prec)
        else:
            s["op"] = mf.heat_operator(ctx, q.heat, phi=f["phi"], precision=prec)
    elif kind in ("heat_conv", "gmres_conv"):
        s["op"] = mf.heat_operator(ctx, q.heat, phi=f["phi"], u0=f["u0"])
    elif kind == "heat_melt":
        s["op"] = mf.heat_operator(ctx, q.heat, phi=f["phi"], T_coef=f["Tc"])
    elif kind in ("oseen", "gmres_oseen"):
        s["op"] = mf.oseen_operator(ctx, q.flow, f["phi"], f["u0"])
    elif kind == "oseen_melt":
        s["op"] = mf.oseen_operator(ctx, q.flow, f["phi"], f["u0"], T_coef=f["Tc"])
    elif kind in ("cg", "mg"):
        s["op"] = mf.heat_operator(ctx, q.heat, phi=f["phi"])
    elif kind == "step":
        s["step"] = autograd.HeatStep(ctx, q.heat)
        s["phi"] = f["phi"].requires_grad_(True)
        s["T_old"] = f["x"].requires_grad_(True)
        s["target"] = 0.999 * f["x"].detach()
    elif kind == "picard":
        s["phi"], s["T_old"], s["params"], s["sources"] = f["phi"], f["Tc"], q.heat, W.SourceParams(terms=7)
    elif kind == "interface":
        s["op"] = mf.heat_operator(ctx, q.heat, phi=f["phi"])
        s["phi"], s["u"], s["T"], s["flow"], s["sources"] = f["phi"], f["u0"], f["T"], q.flow, W.SourceParams()
        s["b"], s["ug"] = torch.empty_like(f["T"]), torch.empty_like(f["u0"])
        s["variant"] = mf.MF_TRANSPORT_LIQUID_EXTENSION if case["form"] == "sine" else mf.MF_TRANSPORT_LOCAL
    if kind in ("cg", "mg", "gmres_oseen", "gmres_conv"):
        s["b"] = mf.operator_apply(s["op"], f["x"], torch.empty_like(f["x"]))
        s["x"] = torch.empty_like(f["x"])
    elif "x" in f and kind != "step":
        s["x"], s["y"] = f["x"], torch.empty_like(f["x"])
    if kind == "mg":
        s["mg"] = mf.Multigrid(s["op"], mf.MGConfig(coarse_cells=case["coarse"], degree=1, auto_levels=True,
                                                    smooth_degree=2))
    return s


def run(s):
    kind, case = s["kind"], s["case"]
    if kind in ("heat", "heat_conv", "heat_melt", "oseen", "oseen_melt"):
        apply = mf.operator_apply_transpose if case["transpose"] else mf.operator_apply
        return apply(s["op"], s["x"], s["y"])
    if kind == "cg":
        mf.cg_solve(s["op"], s["b"], s["x"], case["rtol"], 2000)
        return s["x"]
    if kind == "gmres_oseen":
        mf.gmres_solve(s["op"], s["b"], s["x"], case["rtol"], 2000, precond=mf.MF_PC_BLOCK_JACOBI, restart=30)
        return s["x"]
    if kind == "gmres_conv":
        mf.gmres_solve(s["op"], s["b"], s["x"], case["rtol"], 2000, precond=mf.MF_PC_JACOBI, restart=30)
        return s["x"]
    if kind == "mg":
        mf.mg_cg_solve(s["mg"], s["b"], s["x"], case["rtol"], 200)
        return s["x"]
    if kind == "step":
        T, dT = autograd.heat_step(s["step"], s["T_old"], phi=s["phi"])
        loss = torch.sum((T - s["target"]) ** 2)
        gphi, gold = torch.autograd.grad(loss, (s["phi"], s["T_old"]))
        return {"T": T.detach(), "dT": dT.detach(), "dphi": gphi, "dT_old": gold}
    if kind == "picard":
        return picard.heat_step(s["ctx"], s["params"], s["phi"], s["T_old"], sources=s["sources"]).T
    mf.heat_source_rhs(s["op"], s["sources"], s["T"], s["b"])
    mf.transport_velocity(s["ctx"], s["variant"], s["flow"], s["sources"], s["phi"], s["u"], s["T"], s["ug"])
    return {"b": s["b"], "u_gamma": s["ug"]}


def work(case):
    """Bytes (each input read once, each output written once; a Krylov
    iteration reads and writes its vectors once more) and flops of the
    sum-factorized algorithm."""
    nodes = 1
    for k in ("nx", "ny", "nz"):
        nodes *= 2 * case[k] + 1
    cells = case["nx"] * case["ny"] * case["nz"]
    kind = case["kind"]
    if kind == "heat":
        size = 4 if case["dtype"] == "float32" else 8
        if case["coefficients"] == "points":
            return {"bytes": 2 * size * nodes + 54 * size * cells, "flops": 1458 * cells}
        return {"bytes": 3 * size * nodes, "flops": 1998 * cells}
    if kind == "heat_conv":
        return {"bytes": 48 * nodes, "flops": 3456 * cells}
    if kind == "heat_melt":
        return {"bytes": 32 * nodes, "flops": 3400 * cells}
    if kind in ("oseen", "oseen_melt"):
        return {"bytes": (88 if kind == "oseen_melt" else 80) * nodes, "flops": 1170 * nodes}
    slow = case["dt"] >= 1.0
    if kind == "cg":
        its = 45 if slow else 13  # apply (x, phi, y) and x, r, p read and written, diagonal read
        return {"bytes": its * (24 + 56) * nodes, "flops": its * 1998 * cells}
    if kind in ("gmres_oseen", "gmres_conv"):
        comps, its = (3, 31) if kind == "gmres_oseen" else (1, 35)
        apply = 80 if comps == 3 else 48
        return {"bytes": its * (apply + comps * 8 * 2 * its / 2) * nodes, "flops": its * 3456 * comps * cells}
    if kind == "mg":
        its = 7  # FP64 iteration and a V-cycle of about two FP32 applies
        return {"bytes": its * (24 + 56 + 2 * 24) * nodes, "flops": its * 3 * 1998 * cells}
    if kind == "step":
        return {"bytes": 2 * 40 * 80 * nodes, "flops": 2 * 40 * 1998 * cells}
    if kind == "picard":
        return {"bytes": 2 * 30 * 88 * nodes, "flops": 2 * 30 * 3400 * cells}
    return {"bytes": (24 + 64) * nodes, "flops": 2500 * cells}


# ---------------------------------------------------------------------------
# The same results in plain float64 torch
# ---------------------------------------------------------------------------

_R = math.sqrt(15.0) / 10.0


class Cells:
    """Dense cell tables of Q2 elements with 3 x 3 x 3 Gauss points on a mesh."""

    def __init__(self, q, walls=None):
        n, h = q.mesh.n, q.mesh.h
        self.q, self.n, self.N = q, n, q.N
        t = lambda a: torch.tensor(a, dtype=F64, device=DEV)
        S = t([[0.3 + _R, 0.4, 0.3 - _R], [0.0, 1.0, 0.0], [0.3 - _R, 0.4, 0.3 + _R]])
        G = t([[-1 - 4 * _R, 8 * _R, 1 - 4 * _R], [-1.0, 0.0, 1.0], [-1 + 4 * _R, -8 * _R, 1 + 4 * _R]])
        w = t([5 / 18, 4 / 9, 5 / 18])
        k3 = lambda z, y, x: torch.kron(z, torch.kron(y, x))
        self.V = k3(S, S, S)
        self.D = [k3(S, S, G / h[0]), k3(S, G / h[1], S), k3(G / h[2], S, S)]
        self.W = k3(w, w, w) * (h[0] * h[1] * h[2])
        walls = q.mesh.dirichlet if walls is None else walls
        free = torch.ones(q.N[::-1], dtype=torch.bool, device=DEV)
        for bit, at in enumerate([(2, 0), (2, -1), (1, 0), (1, -1), (0, 0), (0, -1)]):
            if walls >> bit & 1:
                free.select(*at).fill_(False)
        self.free = free.reshape(-1)

    def gather(self, f):
        f = f.reshape(self.N[::-1])
        return f.unfold(0, 3, 2).unfold(1, 3, 2).unfold(2, 3, 2).reshape(-1, 27)

    def scatter(self, e):
        nx, ny, nz = self.n
        e = e.reshape(nz, ny, nx, 27)
        out = torch.zeros(self.N[::-1], dtype=F64, device=DEV)
        for i in range(27):
            a, b, c = i % 3, i // 3 % 3, i // 9
            out[c:c + 2 * nz - 1:2, b:b + 2 * ny - 1:2, a:a + 2 * nx - 1:2] += e[..., i]
        return out.reshape(-1)

    def value(self, f):
        return self.gather(f) @ self.V.T

    def grad(self, f):
        g = self.gather(f)
        return [g @ D.T for D in self.D]


def _heaviside(form, eps, phi):
    """H and dH/dphi."""
    if form == "linear":
        return torch.clamp(0.5 + 0.5 * phi, 0.0, 1.0), 0.5 * ((phi > -1.0) & (phi < 1.0)).to(F64)
    p = torch.clamp(phi, -(1.0 - 1e-15), 1.0 - 1e-15)
    d = 2.0 * eps * torch.atanh(p)
    a = math.pi * d / (3.0 * eps)
    H = torch.where(d <= -3 * eps, 0.0, torch.where(d >= 3 * eps, 1.0, 0.5 + d / (6 * eps) + torch.sin(a) / (2 * math.pi)))
    dH = torch.where(d.abs() >= 3 * eps, 0.0, (1 + torch.cos(a)) / (6 * eps) * 2 * eps / (1 - p * p))
    return H, dH


def _solid(p, T):
    fs = torch.clamp((p.T_liq - T) / (p.T_liq - p.T_sol), 0.0, 1.0)
    return fs, fs * fs * (3.0 - 2.0 * fs)


class Heat:
    """The heat operator with its coefficients at the Gauss points."""

    def __init__(self, case, q, f, Tc=None, mass=True, walls=None):
        self.C, p = Cells(q, walls), q.heat
        C = self.C
        ph = None
        if "kq" in f:
            k, rc = f["kq"].double().reshape(-1, 27), f["rcq"].double().reshape(-1, 27)
        else:
            ph = C.value(f["phi"].double().detach())
            H, dH = _heaviside(case["form"], q.eps, ph)
            k_sl, rc_sl = p.k_l, p.rc_l
            if Tc is not None:
                _, Hs = _solid(p, C.value(Tc))
                k_sl, rc_sl = Hs * p.k_s + (1 - Hs) * p.k_l, Hs * p.rc_s + (1 - Hs) * p.rc_l
            k, rc = H * k_sl + (1 - H) * p.k_g, H * rc_sl + (1 - H) * p.rc_g
            self.H, self.dH = H, dH
        self.am = p.alpha_m if mass else 0.0
        self.cm, self.ck = C.W * self.am * rc, C.W * p.alpha_k * k
        if p.penalty:
            self.cm = self.cm + C.W * p.penalty * self.delta(f, p)
        self.rc = rc
        self.u = [C.value(c) for c in f["u0"].reshape(3, -1)] if "u0" in f else None

    def delta(self, f, p):
        gn = sum(g * g for g in self.C.grad(f["phi"].double().detach())).sqrt()
        return self.dH * gn * (p.rc_g + self.H * (p.rc_l - p.rc_g)) * 3.0 / (p.rc_g ** 2 + p.rc_l * p.rc_g + p.rc_l ** 2)

    def apply(self, x, transpose=False):
        C = self.C
        g = C.gather(torch.where(C.free, x, 0.0))
        v = g @ C.V.T
        mass = self.cm * v
        out = 0.0
        for d in range(3):
            gd = g @ C.D[d].T
            flux = self.ck * gd
            if self.u is not None and transpose:
                flux = flux + C.W * self.rc * self.u[d] * v
            elif self.u is not None:
                mass = mass + C.W * self.rc * self.u[d] * gd
            out = out + flux @ C.D[d]
        return torch.where(C.free, C.scatter(out + mass @ C.V), x)

    def diagonal(self):
        C = self.C
        d = self.cm @ (C.V * C.V) + sum(self.ck @ (D * D) for D in C.D)
        return torch.where(C.free, C.scatter(d), 1.0)

    def solve(self, b, rtol=1e-15, maxit=400):
        """Jacobi-CG down to rounding (the best iterate by its residual)."""
        M = 1.0 / self.diagonal()
        x = torch.zeros_like(b)
        r = b.clone()
        z = M * r
        p, rz, stop = z, r @ z, rtol * float(b.norm())
        for _ in range(maxit):
            q = self.apply(p)
            a = rz / (p @ q)
            x = x + a * p
            r = r - a * q
            if float(r.norm()) <= stop:
                break
            z = M * r
            rz, old = r @ z, rz
            p = z + (rz / old) * p
        return x


def _exact_oseen(case, q, f):
    C, p = Cells(q), q.flow
    H, _ = _heaviside(case["form"], q.eps, C.value(f["phi"]))
    rho_sl, mu_sl, darcy = p.rho_l, p.mu_l, 0.0
    if "Tc" in f:
        fs, Hs = _solid(p, C.value(f["Tc"]))
        rho_sl, mu_sl = Hs * p.rho_s + (1 - Hs) * p.rho_l, Hs * p.mu_s + (1 - Hs) * p.mu_l
        darcy = p.darcy_C * fs * fs / ((1 - fs) ** 3 + p.darcy_b)
    rho = 1.0 / (H / rho_sl + (1 - H) / p.rho_g)
    mu = H * mu_sl + (1 - H) * p.mu_g
    u0 = [C.value(c) for c in f["u0"].reshape(3, -1)]
    x = f["x"].reshape(3, -1)
    xm = [torch.where(C.free, c, 0.0) for c in x]
    val, grad = [C.value(c) for c in xm], [C.grad(c) for c in xm]
    ys = []
    for c in range(3):
        m = C.W * (p.alpha_m * rho + darcy) * val[c]
        out = 0.0
        for d in range(3):
            flux = C.W * p.alpha_v * mu * (grad[c][d] + grad[d][c])
            if case["transpose"]:
                flux = flux + C.W * p.alpha_c * rho * u0[d] * val[c]
            else:
                m = m + C.W * p.alpha_c * rho * u0[d] * grad[c][d]
            out = out + flux @ C.D[d]
        ys.append(torch.where(C.free, C.scatter(out + m @ C.V), x[c]))
    return torch.cat(ys)


def _tanasawa(s):
    rs = 8.314 / s.molar_mass
    return (2 * s.evap_coeff / (2 - s.evap_coeff) * s.h_v / math.sqrt(2 * math.pi * rs) * s.vapor_density /
            (s.T_boil * math.sqrt(s.T_boil)))


def _exact_sources(case, q, f, s, T, A):
    """Right-hand side of the interface heat fluxes."""
    C, p = A.C, q.heat
    g = C.grad(f["phi"])
    gn = sum(v * v for v in g).sqrt()
    ge = sum(s.dir[d] * g[d] for d in range(3))
    drc = A.dH * (p.rc_g + A.H * (p.rc_l - p.rc_g)) * 3.0 / (p.rc_g ** 2 + p.rc_l * p.rc_g + p.rc_l ** 2)
    X = [C.value(q.flat(c.expand(q.N[::-1]))) - s.focus[d] for d, c in enumerate((q.X, q.Y, q.Z))]
    t = sum(X[d] * s.dir[d] for d in range(3))
    d2 = sum((X[d] - t * s.dir[d]) ** 2 for d in range(3))
    peak = 2 * s.absorptivity * s.power / (math.pi * s.radius ** 2)
    src = peak * torch.clamp(ge, min=0.0) * torch.exp(-2 * d2 / s.radius ** 2) * drc
    src = src - _tanasawa(s) * (C.value(T) - s.T_boil) * s.h_v * gn * drc
    if s.terms & 4:
        src = src + p.penalty * s.T_boil * gn * drc
    return torch.where(C.free, C.scatter((C.W * src) @ C.V), 0.0)


def _axis_derivative(d, dim, h):
    """Derivative along an axis at every node, averaged over the cells there."""
    d = d.movedim(dim, 0)
    lo, mid, hi = d[0:-2:2], d[1:-1:2], d[2::2]
    left, right = -3 * lo + 4 * mid - hi, lo - 4 * mid + 3 * hi
    g = torch.zeros_like(d)
    g[1::2] = hi - lo
    g[0:-2:2] += left
    g[2::2] += right
    g[2:-2:2] *= 0.5
    return (g / h).movedim(0, dim)


def _exact_transport(case, q, f, s):
    shape, h = q.N[::-1], q.mesh.h
    p, eps = q.flow, q.eps
    lim = 1.0 - 1e-15
    d = (2 * eps * torch.atanh(torch.clamp(f["phi"], -lim, lim))).reshape(shape)
    g = [_axis_derivative(d, 2 - k, h[k]) for k in range(3)]
    gn = sum(v * v for v in g).sqrt()
    n = [torch.where(gn > 1e-8, v / gn, 0.0) for v in g]
    x = [q.X, q.Y, q.Z]
    u, T = f["u0"].reshape(3, *shape), f["T"].reshape(shape)
    if case["form"] == "linear":
        H = torch.clamp(0.5 + 0.5 * f["phi"].reshape(shape), 0.0, 1.0)
        sp = _tanasawa(s) * (T - s.T_boil) * (H / p.rho_l + (1 - H) / p.rho_g)
        return torch.cat([(u[c] + sp * n[c]).reshape(-1) for c in range(3)])

    def weights(dist):
        at, ws = [], []
        for k in range(3):
            pt = torch.clamp(x[k] + dist * n[k], 0.0, q.hi[k])
            c = torch.clamp(torch.floor(pt / h[k]), 0, q.mesh.n[k] - 1)
            xi = pt / h[k] - c
            at.append(2 * c.long())
            ws.append(((2 * xi - 1) * (xi - 1), 4 * xi * (1 - xi), xi * (2 * xi - 1)))
        return at, ws

    def values(loc, fields):
        (ix, iy, iz), (wx, wy, wz) = loc
        out = [torch.zeros_like(gn) for _ in fields]
        for c in range(3):
            for b in range(3):
                for a in range(3):
                    i = (ix + a) + q.N[0] * ((iy + b) + q.N[1] * (iz + c))
                    w = wx[a] * wy[b] * wz[c]
                    for o, v in zip(out, fields):
                        o += w * v.reshape(-1)[i]
        return out

    mdot = _tanasawa(s) * (values(weights(-d), [T])[0] - s.T_boil)
    base = values(weights(3 * eps - d), list(u))
    return torch.cat([(base[c] + mdot / p.rho_l * n[c]).reshape(-1) for c in range(3)])


def _exact_step(case, q, f):
    phi, T_old = f["phi"], f["x"]
    A = Heat(case, q, {"phi": phi})
    K = Heat(case, q, {"phi": phi}, mass=False, walls=0)
    C, p = A.C, q.heat
    dT = A.solve(torch.where(C.free, -K.apply(T_old), 0.0))
    T = T_old + dT
    gT = 2.0 * (T - 0.999 * T_old)
    lam = A.solve(torch.where(C.free, gT, 0.0))
    dk = -p.alpha_k * C.W * sum(a * b for a, b in zip(C.grad(lam), C.grad(T)))
    drc = -p.alpha_m * C.W * C.value(lam) * C.value(dT)
    dphi = C.scatter((A.dH * ((p.k_l - p.k_g) * dk + (p.rc_l - p.rc_g) * drc)) @ C.V)
    # the loss's own dependence on T_old through its target is not part of the step
    return {"T": T, "dT": dT, "dphi": dphi, "dT_old": gT - K.apply(lam)}


def _exact_picard(case, q, f):
    T_old, s = f["Tc"], W.SourceParams(terms=7)
    T = T_old
    for _ in range(30):
        A = Heat(case, q, f, Tc=T)
        K = Heat(case, q, f, Tc=T, mass=False, walls=0)
        b = _exact_sources(case, q, f, s, T, A)
        new = T_old + A.solve(torch.where(A.C.free, b - K.apply(T_old), 0.0), rtol=1e-14)
        step = float((new - T).norm() / new.norm())
        T = new
        if step <= 1e-10:
            break
    return T


def exact(case, seed):
    q, f = _fields(case, seed)
    kind = case["kind"]
    if kind in ("heat", "heat_conv", "heat_melt"):
        return Heat(case, q, f, Tc=f.get("Tc")).apply(f["x"].double(), case["transpose"])
    if kind in ("oseen", "oseen_melt"):
        return _exact_oseen(case, q, f)
    if kind in ("cg", "mg", "gmres_oseen", "gmres_conv"):
        return f["x"]  # the right-hand side is the operator applied to it
    if kind == "step":
        return _exact_step(case, q, f)
    if kind == "picard":
        return _exact_picard(case, q, f)
    s = W.SourceParams()
    A = Heat(case, q, {"phi": f["phi"]})
    return {"b": _exact_sources(case, q, f, s, f["T"], A), "u_gamma": _exact_transport(case, q, f, s)}
