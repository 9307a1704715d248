"""Measured cases: the work that users of this framework have it do.

A pass is one output interval of a run (step n times, then read the macroscopic fields) or one
gradient through a recorded run.  The cases cover the three 2D stencils and D3Q39, both storage
precisions, the boundary kinds with and without corners, the largest grids of the benchmark, the
small ones of the tests (where launches and latency count), odd sizes, and the single step.
Single-precision storage hands its fields on in single precision.

exact() is the same map in 64 bits in plain torch: stencils from their moment conditions, the
Hermite equilibrium per velocity, one operation at a time; gradients by automatic differentiation.
"""
import itertools
import math

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

from paper_2307_16766_amd import lbm, lbm3d
from paper_2307_16766_amd.autograd import simulate

RELAXED = ("lodi_relax", "cbc_relax")
FULL = ("cbc", "cbc_relax")
CHARACTERISTIC = ("lodi", "lodi_relax", "cbc", "cbc_relax")


# ---------------------------------------------------------------------------- the cases
def forward(name, q, size, bc, flow, steps, precision="fp64", recon="equilibrium", watch=False, axis=0):
    """One output interval of a run: bc = sides x0, x1, y0, y1 (2D) or the two faces (3D)."""
    nx, ny, nz = tuple(size) + (1,) * (3 - len(size))
    return dict(name=name, kind="forward", q=q, nx=nx, ny=ny, nz=nz, bc=",".join(bc), flow=flow, steps=steps,
                precision=precision, recon=recon, watch=watch, axis=axis)


def gradient(name, q, size, bc, flow, steps, every):
    """One gradient of a loss of the final fields with respect to the initial ones, sigma and alpha."""
    return dict(name=name, kind="gradient", q=q, nx=size[0], ny=size[1], nz=1, bc=",".join(bc), flow=flow, steps=steps,
                every=every, precision="fp64", recon="equilibrium", watch=False, axis=0)


def listed():
    four = ["lodi_relax"] * 4
    return [
        # a temperature step leaving a short strip, looked at after every step: the smallest call
        forward("front_q17_200x20", 17, (200, 20), ["cbc", "cbc", "periodic", "periodic"], "front", 1),
        # isothermal pulse between two relaxed sides
        forward("pulse_q9_256x128", 9, (256, 128), ["lodi_relax", "lodi_relax", "periodic", "periodic"], "pulse", 10),
        # fluid at rest in an open box with corners, its totals watched (the grid of the gradient workload)
        forward("rest_q37_256x256", 37, (256, 256), four, "rest", 10, watch=True),
        # thermal pulse leaving an open box, single-precision storage
        forward("pulse_q37_512x512_f32", 37, (512, 512), four, "pulse", 20, "fp32dev"),
        # vortex carried through a relaxed outflow, a middle-sized grid with odd sizes
        forward("vortex_q37_1023x509", 37, (1023, 509), ["lodi_relax", "cbc_relax", "periodic", "periodic"], "vortex", 20),
        # the extended periodic grid that boundary errors are measured against
        forward("reference_q17_1950x1950", 17, (1950, 1950), ["periodic"] * 4, "vortex", 20),
        # the throughput run of the benchmark: inlet, relaxed outflow
        forward("shear_q37_4096x2048_f32", 37, (4096, 2048), ["dirichlet", "lodi_relax", "periodic", "periodic"], "shear", 20,
                "fp32dev"),
        # the same flow in double precision between walls of every kind of reconstruction, odd sizes
        forward("shear_q37_2047x1301", 37, (2047, 1301), ["lodi_relax", "cbc_relax", "periodic", "periodic"], "shear", 10,
                recon="neep"),
        # gradient through a recorded run in an open box with corners
        gradient("gradient_q37_256x256", 37, (256, 256), four, "drift", 60, 30),
        # gradient on a small odd grid, relaxed outflow, several checkpoints
        gradient("gradient_q17_131x75", 17, (131, 75), ["lodi_relax", "cbc_relax", "periodic", "periodic"], "drift", 40, 15),
        # three dimensions at the size of the benchmark, single-precision storage
        forward("box_q39_512x256x256_f32", 39, (512, 256, 256), ["lodi_relax", "cbc_relax"], "pulse", 5, "fp32dev"),
        # a small odd duct with its faces along y
        forward("duct_q39_61x90x47", 39, (61, 90, 47), ["lodi_relax", "cbc_relax"], "pulse", 5, axis=1),
    ]


def draw(rng):
    def between(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["forward", "forward", "forward", "gradient", "forward3"])
    x_sides = rng.choice([["lodi_relax", "cbc_relax"], ["lodi", "lodi_relax"], ["lodi_relax", "lodi_relax"],
                          ["dirichlet", "lodi_relax"]])
    if kind == "gradient":
        q = rng.choice([17, 37])
        bc = rng.choice([["lodi_relax"] * 4, x_sides + ["periodic", "periodic"]])
        c = gradient("", q, (between(40, 300), between(40, 300)), bc, "drift", rng.randint(15, 60), rng.randint(10, 40))
    elif kind == "forward3":
        nx, ny, nz = between(20, 400), between(8, 250), between(8, 250)
        faces = rng.choice([["lodi_relax", "cbc_relax"], ["lodi", "lodi_relax"], ["periodic", "periodic"]])
        axis = rng.randint(0, 2)
        size = [(nx, ny, nz), (nz, nx, ny), (ny, nz, nx)][axis]
        c = forward("", 39, size, faces, "pulse", rng.randint(1, 8), rng.choice(["fp64", "fp32dev"]), axis=axis)
    else:
        q = rng.choice([9, 17, 37, 37, 37])
        nx, ny = between(40, 4000), between(20, 2000)
        if q == 9:
            x_sides = rng.choice([["lodi_relax", "lodi_relax"], ["lodi", "lodi_relax"], ["dirichlet", "lodi_relax"]])
        bc = rng.choice([x_sides + ["periodic", "periodic"], x_sides + ["periodic", "periodic"], ["lodi_relax"] * 4,
                         ["periodic"] * 4])
        flow = "pulse" if bc[2] != "periodic" else rng.choice(["pulse", "vortex", "shear"])
        recon = rng.choice(["equilibrium", "neep"]) if bc[0] in CHARACTERISTIC else "equilibrium"
        c = forward("", q, (nx, ny), bc, flow, rng.randint(1, 20), rng.choice(["fp64", "fp32dev"]), recon)
    c.pop("name")
    return c


def relaxation(case):
    """Relaxation settings of every relaxed side (transverse relaxation only without corners)."""
    corners = "periodic" not in case["bc"] and case["q"] != 39
    return dict(sigma=0.25, alpha=0.0 if corners or case["q"] == 9 else 0.1, mach=0.05)


def tau_of(case):
    """nu = 0.1 on D2Q37, the relaxation times of the other stencils' workloads."""
    return {9: 0.6, 17: 0.9, 37: 0.5 + 0.1 / stencil(37)[2], 39: 0.7}[case["q"]]


# ---------------------------------------------------------------------------- inputs
def fields_of(case, seed):
    """Initial (rho, u_x, u_y[, u_z], T) on the GPU, and the inlet profile [ny][4] of a Dirichlet side."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(int(seed))
    kw = dict(dtype=torch.float64, device=dev)
    nx, ny, nz, q = case["nx"], case["ny"], case["nz"], case["q"]
    d = 3 if q == 39 else 2
    shape = (nz, ny, nx)[3 - d:]
    ax = [torch.arange(n, **kw) for n in shape]
    at = torch.rand(3, generator=g, **kw)

    def noise(a):
        return a * (2.0 * torch.rand(shape, generator=g, **kw) - 1.0)

    def squared_distance():
        r2 = torch.zeros(shape, **kw)
        for k in range(d):
            x = (ax[k] - (0.3 + 0.4 * at[k]) * (shape[k] - 1)).reshape([-1 if j == k else 1 for j in range(d)])
            r2 = r2 + x * x
        return r2

    cs = math.sqrt(stencil(q)[2])
    rho, T = torch.ones(shape, **kw), torch.ones(shape, **kw)
    u = [torch.zeros(shape, **kw) for _ in range(d)]
    inlet = None
    flow = case["flow"]
    if flow == "pulse":       # pressure pulse in a fluid at rest (a slow oblique stream in three dimensions)
        p = 1e-3 * torch.exp(-squared_distance() / (2.0 * (0.06 * min(shape) + 4.0) ** 2))
        if q == 9:
            rho = rho + p
        else:
            T = T + p
        if d == 3:
            u = [x + 0.02 - 0.005 * k for k, x in enumerate(u)]
    elif flow == "rest":      # thermal noise
        T = T + 1e-4 * torch.randn(shape, generator=g, **kw)
    elif flow == "drift":     # warm fluid, a pulse and thermal noise in a slow meandering oblique stream
        p = torch.exp(-squared_distance() / (2.0 * (0.06 * min(shape) + 4.0) ** 2))
        T = T + 2e-3 + 1e-3 * p + 1e-4 * torch.randn(shape, generator=g, **kw)
        ph = 2.0 * math.pi * (ax[1][None, :] / nx + ax[0][:, None] / ny)
        u = [0.02 + 0.01 * torch.cos(ph), 0.015 + 0.01 * torch.sin(ph)]
    elif flow == "vortex":    # isentropic vortex in a stream of Mach 0.2
        x0, y0, R, s = (0.3 + 0.4 * at[0]) * nx, (0.3 + 0.4 * at[1]) * ny, 20.0, 0.05
        dx, dy = ax[1][None, :] - x0, ax[0][:, None] - y0
        e = torch.exp(1.0 - (dx * dx + dy * dy) / R ** 2)
        amp = s * torch.sqrt(e) / R
        u = [0.2 * cs - amp * dy, amp * dx]
        if q != 9:
            T = 1.0 - s ** 2 / (4.0 * cs * cs) * e
        rho = 1.0 - s ** 2 / (4.0 * cs * cs) * e
    elif flow == "shear":     # shear layer with noise and a slow stream across it
        base = 0.1 * torch.tanh((ax[0] - (0.4 + 0.2 * at[0]) * ny) / 10.0)
        u = [base[:, None] + noise(1e-3), 0.01 + noise(1e-3)]
        inlet = torch.stack([torch.ones_like(base), base, torch.full_like(base, 0.01), torch.ones_like(base)], dim=1)
    elif flow == "front":     # warm slab between two smooth fronts in a stream of Mach 0.1
        x = ax[1] - (at[0] - 0.5) * 0.1 * nx
        T = T + 2.5e-4 * (torch.tanh(0.5 * (x - nx / 4)) - torch.tanh(0.5 * (x - 3 * nx / 4)))[None, :]
        u = [u[0] + 0.1 * cs + noise(1e-4), u[1] + noise(1e-4)]
    if inlet is None and "dirichlet" in case["bc"]:
        inlet = torch.stack([f[:, 0].clone() for f in (rho, u[0], u[1], T)], dim=1)
    return [rho, *u, T], inlet


def prepare(case, seed):
    fields, inlet = fields_of(case, seed)
    bc = case["bc"].split(",")
    if case["kind"] == "gradient":
        g = torch.Generator(device="cuda").manual_seed(int(seed) + 7)
        leaves = [torch.tensor(v, dtype=torch.float64, device="cuda", requires_grad=True) for v in gradient_parameters(case)]
        leaves += [f.requires_grad_(True) for f in fields]
        weights = 0.5 + torch.rand((4, case["ny"], case["nx"]), dtype=torch.float64, device="cuda", generator=g)
        return dict(case=case, leaves=leaves, cotangent=weights)   # of a weighted mean of the final fields
    if case["q"] == 39:
        sim = lbm3d.LBM3D(case["nx"], case["ny"], case["nz"], tau_of(case), bc, fields, precision=case["precision"],
                          axis=case["axis"])
    else:
        sim = lbm.LBM(case["q"], case["nx"], case["ny"], tau_of(case), bc, fields, precision=case["precision"])
    for s, b in enumerate(bc):
        if b in RELAXED:
            sim.set_relax(s, **relaxation(case))
    if inlet is not None and "dirichlet" in bc:
        sim.set_inlet(bc.index("dirichlet"), inlet.cpu().numpy())
    if case["recon"] != "equilibrium":
        sim.set_reconstruction(-1, case["recon"])
    return dict(case=case, sim=sim)


def gradient_parameters(case):
    r = relaxation(case)
    return r["sigma"], r["alpha"]


# ---------------------------------------------------------------------------- one pass
def run(state):
    case = state["case"]
    if case["kind"] == "gradient":
        out = simulate(*state["leaves"], stencil=case["q"], nx=case["nx"], ny=case["ny"], tau=tau_of(case),
                       bc=case["bc"].split(","), nsteps=case["steps"], every=case["every"],
                       relax=dict(mach=relaxation(case)["mach"]))
        return [out.detach(), *torch.autograd.grad(out, state["leaves"], state["cotangent"])]
    sim = state["sim"]
    sim.step(case["steps"])
    out = sim.macroscopic()
    if case["precision"] == "fp32dev":
        out = [f.float() for f in out]
    if case["watch"]:
        out.append(sim.diagnostics()[:7])
    return out


def work(case):
    """The state read and written once, the fields written; a gradient reads each step's moments back.
    Operations per node and step: moments, equilibrium and relaxation of q populations (about ten
    each), about three times as many for a step's reverse."""
    n, q, steps = case["nx"] * case["ny"] * case["nz"], case["q"], case["steps"]
    size = 8 if case["precision"] == "fp64" else 4
    d = 3 if q == 39 else 2
    if case["kind"] == "gradient":
        return dict(bytes=n * (2.0 * q * 8 + 2 * 4 * 8 * steps + 8 * 4 * 8), flops=40.0 * q * n * steps)
    out = (d + 2) * n * size
    return dict(bytes=2.0 * q * n * size + out, flops=10.0 * q * n * steps)


# ---------------------------------------------------------------------------- 64-bit reference
GROUPS = {9: ([(0, 0), (1, 0), (1, 1)], 1 / 3, 2),
          17: ([(0, 0), (1, 0), (1, 1), (2, 2), (3, 0)], 72 / (5 * (25 + math.sqrt(193))), 3),
          37: ([(0, 0), (1, 0), (1, 1), (2, 0), (2, 1), (2, 2), (3, 0), (3, 1)], None, 4),
          39: ([(0, 0, 0), (1, 0, 0), (1, 1, 1), (2, 0, 0), (2, 2, 0), (3, 0, 0)], 2 / 3, 3)}
_stencils = {}


def stencil(q):
    """(velocities, weights, cs^2, order of the equilibrium, layers M): the weights make the discrete
    moments of the velocity groups those of a Gaussian."""
    if q in _stencils:
        return _stencils[q]
    groups, cs2, order = GROUPS[q]
    if cs2 is None:   # the real root of 35 s^3 - 70 s^2 + 49 s - 12
        cs2 = 0.7
        for _ in range(50):
            cs2 -= (35 * cs2 ** 3 - 70 * cs2 ** 2 + 49 * cs2 - 12) / (105 * cs2 ** 2 - 140 * cs2 + 49)
    d = len(groups[0])
    members = [sorted({tuple(s * c for s, c in zip(sg, p)) for p in itertools.permutations(g)
                       for sg in itertools.product((1, -1), repeat=d)}) for g in groups]
    gauss = {0: 1, 2: 1, 4: 3, 6: 15, 8: 105}
    degree = {9: 4, 17: 6, 37: 8, 39: 6}[q]
    rows, rhs = [], []
    for e in itertools.product(range(0, degree + 1, 2), repeat=d):
        if sum(e) <= degree:
            rows.append([sum(math.prod(c ** k for c, k in zip(v, e)) for v in m) / cs2 ** (sum(e) / 2) for m in members])
            rhs.append(math.prod(gauss[k] for k in e))
    w = np.linalg.lstsq(np.array(rows, float), np.array(rhs, float), rcond=None)[0]
    c = [v for m in members for v in m]
    ws = [float(x) for x, m in zip(w, members) for _ in m]
    _stencils[q] = (c, ws, cs2, order, 1 if q == 9 else 3)
    return _stencils[q]


class Reference:
    """The time step in plain torch.  Arrays have their axes as (z,) y, x; velocity component k
    belongs to axis x, y, z.  Populations are kept as deviations from the weights, [q, ...]."""

    def __init__(self, case, fields, inlet, sigma, alpha):
        self.q = case["q"]
        self.c, self.w, self.cs2, self.order, self.M = stencil(self.q)
        self.thermal = self.q != 9
        self.d = len(self.c[0])
        self.omega, self.nu = 1.0 / tau_of(case), (tau_of(case) - 0.5) * self.cs2
        self.MS = 2 if self.M == 1 else 1
        self.gamma = 1.0 + 2.0 / self.d
        self.neep = case["recon"] == "neep"
        self.shape = tuple(fields[0].shape)
        bc = case["bc"].split(",")
        axes = [case["axis"]] if self.d == 3 else [0, 1]
        kinds = dict(zip([(a, e) for a in axes for e in (-1, 1)], bc))
        self.sides = [(a, e, b) for (a, e), b in kinds.items() if b != "periodic"]   # component axis, outward, kind
        self.open = {a for a, _, _ in self.sides}
        self.corners = len(self.open) == 2
        r = relaxation(case)
        cinf = math.sqrt(self.gamma * self.cs2 if self.thermal else self.cs2)
        self.alpha, self.sigma = alpha, sigma
        self.K = {a: sigma * (1 - r["mach"] ** 2) * cinf / self.shape[self.dim(a)] for a in self.open}
        U = torch.stack(fields, dim=-1)
        if not self.thermal:
            U = torch.cat([U[..., :-1], torch.ones_like(U[..., -1:])], dim=-1)
        self.inlet = inlet
        self.f = self.equilibrium(U)
        self.state = []
        for a, e, b in self.sides:
            if b == "dirichlet":
                self.lay(self.f, a, e, self.equilibrium(self.profile()))
            st = {}
            if b in CHARACTERISTIC:
                st["U"] = self.local(torch.stack([self.rows(U, a, e, -j) for j in range(1, self.M + 1)]), a, e)
                st["X"] = self.local(torch.stack([self.rows(U, a, e, k) for k in range(self.MS)]), a, e)
                if b in FULL:
                    z = torch.stack([self.rows(U, a, e, self.M + k) for k in range(3)])[..., :1]
                    st["vis"] = torch.cat([z, torch.zeros(z.shape[:-1] + (self.d * (self.d + 1) // 2 + self.d,),
                                                          dtype=z.dtype, device=z.device)], dim=-1)
            self.state.append(st)
        if self.corners:
            self.cU, self.cD = self.corner_nodes(U, 0), torch.stack([self.corner_nodes(U, 1), self.corner_nodes(U, 2)])

    # geometry: index of the node k steps inward of x_f (k < 0: the layers) on the axis of a side
    def dim(self, a):
        return self.d - 1 - a

    def index(self, a, e, k):
        return self.M + k if e < 0 else self.shape[self.dim(a)] - 1 - self.M - k

    def cut(self, U, a):
        """Rows of a side: the nodes along it without the corner blocks."""
        if self.corners:
            dim = 0   # the remaining axis
            return U.narrow(dim, self.M, U.shape[dim] - 2 * self.M)
        return U

    def rows(self, U, a, e, k):
        return self.cut(U.select(self.dim(a), self.index(a, e, k)), a)

    def local(self, U, a, e):
        """(rho, u_n, u_t.., T) of a side: outward normal velocity, tangential ones in cyclic order."""
        return torch.stack([U[..., 0], e * U[..., 1 + a]] + [U[..., 1 + (a + k) % self.d] for k in range(1, self.d)]
                           + [U[..., -1]], dim=-1)

    def world(self, U, a, e):
        comp = {a: e * U[..., 1]}
        for k in range(1, self.d):
            comp[(a + k) % self.d] = U[..., 1 + k]
        return torch.stack([U[..., 0]] + [comp[k] for k in range(self.d)] + [U[..., -1]], dim=-1)

    def profile(self):
        p = self.inlet
        return p if self.thermal else torch.cat([p[..., :-1], torch.ones_like(p[..., -1:])], dim=-1)

    # node physics
    def moments(self, g):
        m = [0.0] * (self.d + 2)   # sum g, sum g c, sum g |c|^2
        for p, c in zip(g, self.c):
            for k, v in enumerate((1,) + c + (sum(x * x for x in c),)):
                if v:
                    m[k] = m[k] + v * p
        rho = 1.0 + m[0]
        u = [m[1 + k] / rho for k in range(self.d)]
        T = torch.ones_like(rho)
        if self.thermal:
            j2 = sum(m[1 + k] * u[k] for k in range(self.d))
            T = 1.0 + (m[-1] - j2 - self.d * self.cs2 * m[0]) / (self.d * self.cs2 * rho)
        return torch.stack([rho, *u, T], dim=-1)

    def equilibrium(self, U):
        rho, th, d = U[..., 0], U[..., -1] - 1.0, self.d
        u = [U[..., 1 + k] for k in range(d)]
        u2 = sum(x * x for x in u) / self.cs2
        out = torch.empty((self.q,) + tuple(rho.shape), dtype=rho.dtype, device=rho.device)
        planes = []
        for c, w in zip(self.c, self.w):
            a = sum(k * x for k, x in zip(c, u) if k) if any(c) else torch.zeros_like(rho)
            a = a / self.cs2
            xi2 = sum(k * k for k in c) / self.cs2
            h = a + 0.5 * (a * a - u2 + th * (xi2 - d))
            if self.order >= 3:
                h = h + a / 6 * (a * a - 3 * u2 + 3 * th * (xi2 - d - 2))
            if self.order >= 4:
                h = h + (a ** 4 - 6 * a * a * u2 + 3 * u2 * u2 + 6 * th * (a * a * (xi2 - d - 4) + u2 * (d + 2 - xi2))
                         + 3 * th * th * (xi2 * xi2 - 2 * (d + 2) * xi2 + d * (d + 2))) / 24
            p = w * ((rho - 1.0) + rho * h)
            if p.requires_grad:
                planes.append(p)
            else:
                out[len(planes)] = p
                planes.append(None)
        return torch.stack(planes) if planes[0] is not None else out

    def pull(self, f):
        return torch.stack([torch.roll(f[i], tuple(self.c[i][self.d - 1 - k] for k in range(self.d)), tuple(range(self.d)))
                            for i in range(self.q)])

    def lay(self, f, a, e, values, layer=None):
        """Set a side's layers (all, or one) to the populations `values` [q, rows]."""
        dim = 1 + self.dim(a)
        for j in ([layer] if layer else range(1, self.M + 1)):
            s = f.select(dim, self.index(a, e, -j))
            (s.narrow(1, self.M, s.shape[1] - 2 * self.M) if self.corners else s).copy_(values)

    # viscous terms of a CBC side (no corners next to it)
    def viscous_moments(self, g, U, a, e):
        fn = g - self.equilibrium(U)
        fac = 1.0 - 0.5 * self.omega
        order = [a] + [(a + k) % self.d for k in range(1, self.d)]
        sign = [e] + [1] * (self.d - 1)
        c = torch.tensor([[v[o] * s for o, s in zip(order, sign)] for v in self.c], dtype=g.dtype, device=g.device)
        w = torch.tensor(self.w, dtype=g.dtype, device=g.device).reshape((-1,) + (1,) * (g.dim() - 1))
        u = [s * U[..., 1 + o] for o, s in zip(order, sign)]

        def per(k):
            return c[:, k].reshape((-1,) + (1,) * (g.dim() - 1))

        P = [-fac * (per(i) * per(j) * fn).sum(0) for i in range(self.d) for j in range(i, self.d)]
        rel = [per(k) - u[k] for k in range(self.d)]
        en = (w + g) * sum(x * x for x in rel)
        qf = [0.5 * fac * (en * x).sum(0) for x in rel]
        return torch.stack([U[..., 0]] + P + qf, dim=-1)

    def viscous_terms(self, vis):
        d = self.d
        pair = {}
        for n, (i, j) in enumerate((i, j) for i in range(d) for j in range(i, d)):
            pair[i, j] = pair[j, i] = 1 + n
        heat0 = 1 + d * (d + 1) // 2

        def along(k, m):   # derivative of moment m along local axis k
            v = vis[..., m]
            return 0.5 * (3 * v[0] - 4 * v[1] + v[2]) if k == 0 else self.difference(v[0], k, 1)

        rho = vis[0][..., 0]
        V = [torch.zeros_like(rho)]
        V += [sum(along(j, pair[i, j]) for j in range(d)) / rho for i in range(d)]
        pp = sum(vis[0][..., pair[i, j]] ** 2 for i in range(d) for j in range(d))
        div = sum(along(j, heat0 + j) for j in range(d))
        if d == 2:   # the heating of a plane flow
            v0 = vis[0]
            heat = (0.5 * (v0[..., 1] ** 2 + v0[..., 3] ** 2) + v0[..., 2] ** 2) / (rho * rho * self.nu * self.cs2)
            V.append(-div / (rho * self.cs2) + heat)
        else:
            V.append((-div + pp / (2 * rho * self.nu)) / (rho * 1.5 * self.cs2))
        return torch.stack(V, dim=-1)

    # rows of a side: local tangential axis k = 1.. is axis (a + k) % d, whose array dimension among
    # the side's rows is found from the order z, y, x without the normal axis
    def difference(self, v, k, lead, ends=None):
        dim = self.row_dim[k] + lead - 1
        if ends is not None:
            lo, hi = ends
            v = torch.cat([lo, v, hi], dim=dim)
            n = v.shape[dim] - 2
            return 0.5 * (v.narrow(dim, 2, n) - v.narrow(dim, 0, n))
        return 0.5 * (torch.roll(v, -1, dim) - torch.roll(v, 1, dim))

    def rate(self, U, dn, dt, V, U0, kind, K, alpha):
        """dU/dt of the characteristic system; dt(v) = [d v / d t_1, ..] of a function of the node values."""
        cs2, d, gm = self.cs2, self.d, self.gamma
        rho, un, T, ut = U[..., 0], U[..., 1], U[..., -1], [U[..., 2 + k] for k in range(d - 1)]
        full, relax = kind in FULL, kind in RELAXED
        Pinf = cs2
        tr = range(d - 1)
        Tt = [-sum(dt(lambda W, k=k: W[..., 0] * W[..., 2 + k], k) for k in tr),
              -sum(ut[k] * dt(lambda W: W[..., 1], k) for k in tr)]
        for m in tr:
            p = dt((lambda W: W[..., 0] * W[..., -1]) if self.thermal else (lambda W: W[..., 0]), m)
            Tt.append(-cs2 / rho * p - sum(ut[k] * dt(lambda W, m=m: W[..., 2 + m], k) for k in tr))
        if not self.thermal:
            Tt.append(torch.zeros_like(rho))
        elif d == 2:
            Tt.append(-dt(lambda W: W[..., -1] * W[..., 2], 0))
        else:
            Tt.append(-(gm - 1) * T * sum(dt(lambda W, k=k: W[..., 2 + k], k) for k in tr)
                      - sum(ut[k] * dt(lambda W: W[..., -1], k) for k in tr))
        u0 = U0[..., 1]
        zero = torch.zeros_like(rho)
        if not self.thermal:
            c = math.sqrt(cs2)
            L0 = un * dn[..., 2]
            Lm = (un - c) * (cs2 * dn[..., 0] - rho * c * dn[..., 1])
            Lp = (un + c) * (cs2 * dn[..., 0] + rho * c * dn[..., 1])
            im = ip = zero
            if relax:
                pr = K * (cs2 * rho - Pinf)
                im, ip = pr - alpha * (cs2 * Tt[0] - rho * c * Tt[1]), pr - alpha * (cs2 * Tt[0] + rho * c * Tt[1])
            B0 = torch.where(u0 >= 0, L0, zero)
            Bm, Bp = torch.where(u0 - c >= 0, Lm, im), torch.where(u0 + c >= 0, Lp, ip)
            return torch.stack([-(Bm + Bp) / (2 * cs2), (Bm - Bp) / (2 * c * rho), -B0, zero], dim=-1)
        s, s0 = torch.sqrt(gm * cs2 * T), torch.sqrt(gm * cs2 * U0[..., -1])
        h = (gm - 1) / (2 * gm)
        b = h * s / cs2
        er = T / rho

        def S(x):
            return [-2 * h * er * x[0] + x[-1] / gm] + list(x[2:-1]) + [h * er * x[0] - b * x[1] + h * x[-1],
                                                                       h * er * x[0] + b * x[1] + h * x[-1]]

        Sd, ST = S([dn[..., k] for k in range(d + 2)]), S(Tt)
        lam, lam0 = [un] * d + [un - s, un + s], [u0] * d + [u0 - s0, u0 + s0]
        inc = S([t + V[..., k] for k, t in enumerate(Tt)]) if full else [zero] * (d + 2)
        if relax:
            pr = K * (rho * cs2 * T - Pinf) * h / (rho * cs2)
            inc = inc[:-2] + [inc[-2] + pr - alpha * ST[-2], inc[-1] + pr - alpha * ST[-1]]
        B = [torch.where(l0 >= 0, l * x, i) for l0, l, x, i in zip(lam0, lam, Sd, inc)]
        ac = B[-2] + B[-1]
        rates = [rho / T * (B[0] - ac / (gm - 1)), (B[-2] - B[-1]) / (2 * b)] + [-x for x in B[1:-2]] + [-(B[0] + ac)]
        if full:
            rates = [r + t + V[..., k] for k, (r, t) in enumerate(zip(rates, Tt))]
        return torch.stack(rates, dim=-1)

    def rk4(self, U, inputs, rate):
        """One classical step; inputs(theta) interpolates the outer values in time."""
        acc, k = U, 0.0
        for th, b in ((0.0, 1.0), (0.5, 2.0), (0.5, 2.0), (1.0, 1.0)):
            k = rate(U + th * k, inputs(th))
            acc = acc + b / 6 * k
        return acc

    # corners: order (x0,y0), (x1,y0), (x0,y1), (x1,y1)
    def corner_nodes(self, U, k):
        pts = [(self.index(0, ex, k - 1), self.index(1, ey, k - 1)) for ey in (-1, 1) for ex in (-1, 1)]
        return torch.stack([U[y, x] for x, y in pts])

    def corner_step(self, Dn, Dp):
        n = torch.tensor([[ex, ey] for ey in (-1, 1) for ex in (-1, 1)], dtype=Dn.dtype, device=Dn.device) / math.sqrt(2)

        def loc(U):
            return torch.stack([U[..., 0], U[..., 1] * n[:, 0] + U[..., 2] * n[:, 1],
                                -U[..., 1] * n[:, 1] + U[..., 2] * n[:, 0], U[..., 3]], dim=-1)

        U0 = loc(self.cU)
        kinds = [b for a, e, b in self.sides if a == 0]
        relax = torch.tensor([1.0 if kinds[i % 2] in RELAXED else 0.0 for i in range(4)], dtype=Dn.dtype, device=Dn.device)

        def rate(Y, D):
            dn = (3 * Y - 4 * D[0] + D[1]) / (2 * math.sqrt(2))
            return self.rate(Y, dn, lambda fn, k: torch.zeros_like(Y[..., 0]), None, U0, "lodi_relax", relax * self.K[0], 0.0)

        dn_, dp_ = loc(Dn), loc(Dp)
        R = self.rk4(U0, lambda th: (1 - th) * dn_ + th * dp_, rate)
        return torch.stack([R[..., 0], R[..., 1] * n[:, 0] - R[..., 2] * n[:, 1], R[..., 1] * n[:, 1] + R[..., 2] * n[:, 0],
                            R[..., 3]], dim=-1)

    def side_step(self, st, a, e, kind, Xn, corners):
        dims = [self.dim(k) for k in range(self.d)]
        left = sorted(dims[k] for k in range(self.d) if k != a)
        self.row_dim = {k: left.index(dims[(a + k) % self.d]) for k in range(1, self.d)}
        V = self.viscous_terms(st["vis"]) if kind in FULL else None
        U0, X0, M = st["U"], st["X"], self.M
        alpha = self.alpha if kind in RELAXED else 0.0
        K = self.K[a]

        def inputs(th):
            X = (1 - th) * X0 + th * Xn
            return X, [self.local((1 - th) * o + th * n, a, e) for o, n in corners] if corners else None

        def rate(Y, given):
            X, ends = given
            lad = torch.cat([X.flip(0), Y])   # inner strip node .. x_f, layers 1 .. M
            n = self.MS
            dn = [0.5 * (lad[n + j + 1] - lad[n + j - 1]) for j in range(M - 1)]
            dn.append(0.5 * (3 * lad[n + M - 1] - 4 * lad[n + M - 2] + lad[n + M - 3]))

            def dt(fn, k):
                if ends is None:
                    return self.difference(fn(Y), k + 1, 2)
                return self.difference(fn(Y), k + 1, 2, [fn(c).reshape(1, 1).expand(M, 1) for c in ends])

            return self.rate(Y, torch.stack(dn), dt, V, U0, kind, K, alpha)

        return self.rk4(U0, inputs, rate)

    def step(self):
        g = self.pull(self.f)
        U = self.moments(g)
        f = g + self.omega * (self.equilibrium(U) - g)
        old = self.cU if self.corners else None
        if self.corners:
            D = torch.stack([self.corner_nodes(U, 1), self.corner_nodes(U, 2)])
            self.cU = self.corner_step(self.cD, D)
            self.cD = D
        new = []
        for (a, e, kind), st in zip(self.sides, self.state):
            if kind == "dirichlet":
                self.lay(f, a, e, self.equilibrium(self.profile()))
                new.append(st)
                continue
            Xn = self.local(torch.stack([self.rows(U, a, e, k) for k in range(self.MS)]), a, e)
            ends = None
            if self.corners:   # the corners before the first and after the last row of the side
                pick = [(0, 2), (1, 3), (0, 1), (2, 3)][2 * a + (e > 0)]
                ends = [(old[i], self.cU[i]) for i in pick]
            Ub = self.side_step(st, a, e, kind, Xn, ends)
            nst = dict(U=Ub, X=Xn)
            gdim = 1 + self.dim(a)
            if kind in FULL:
                nst["vis"] = torch.stack([self.viscous_moments(g.select(gdim, self.index(a, e, self.M + k)),
                                                               U.select(self.dim(a), self.index(a, e, self.M + k)), a, e)
                                          for k in range(3)])
            rest = 0.0
            if self.neep:
                gf = g.select(gdim, self.index(a, e, 0))
                gf = gf.narrow(1, self.M, gf.shape[1] - 2 * self.M) if self.corners else gf
                rest = (1 - self.omega) * (gf - self.equilibrium(self.rows(U, a, e, 0)))
            for j in range(1, self.M + 1):
                self.lay(f, a, e, self.equilibrium(self.world(Ub[j - 1], a, e)) + rest, layer=j)
            new.append(nst)
        if self.corners:
            fe = self.equilibrium(self.cU)
            for i, (ey, ex) in enumerate((ey, ex) for ey in (-1, 1) for ex in (-1, 1)):
                for jy, jx in itertools.product(range(1, self.M + 1), repeat=2):
                    f[:, self.index(1, ey, -jy), self.index(0, ex, -jx)] = fe[:, i]
        self.f, self.state = f, new

    # the whole state as a flat list of tensors, for checkpointed automatic differentiation
    def pack(self):
        out = [self.f] + [st[k] for st in self.state for k in sorted(st)]
        return out + ([self.cU, self.cD] if self.corners else [])

    def unpack(self, ts):
        ts = list(ts)
        self.f = ts.pop(0)
        self.state = [{k: ts.pop(0) for k in sorted(st)} for st in self.state]
        if self.corners:
            self.cU, self.cD = ts


def exact(case, seed):
    fields, inlet = fields_of(case, seed)
    if case["kind"] == "gradient":
        st = prepare(case, seed)
        leaves = st["leaves"]
        if inlet is not None:   # an inlet that no profile was given for holds the initial state of its first layer
            inlet = torch.stack([x[:, stencil(case["q"])[4] - 1] for x in leaves[2:]], dim=1)
        ref = Reference(case, leaves[2:], inlet, leaves[0], leaves[1])
        keep = [{k: None for k in s} for s in ref.state]
        ts = ref.pack()

        def one(sigma, alpha, *ts):
            ref.state = keep
            ref.sigma, ref.alpha = sigma, alpha
            r = relaxation(case)
            ref.K = {a: sigma * (1 - r["mach"] ** 2) * math.sqrt(ref.gamma * ref.cs2) / ref.shape[ref.dim(a)] for a in ref.open}
            ref.unpack(ts)
            ref.step()
            return tuple(ref.pack())

        for _ in range(case["steps"]):
            ts = checkpoint(one, leaves[0], leaves[1], *ts, use_reentrant=False)
        out = ref.moments(ts[0]).movedim(-1, 0)
        grads = torch.autograd.grad(out, leaves, st["cotangent"], allow_unused=True)
        return [out.detach(), *[torch.zeros_like(x) if g is None else g for g, x in zip(grads, leaves)]]
    with torch.no_grad():
        r = relaxation(case)
        ref = Reference(case, fields, inlet, r["sigma"], r["alpha"])
        for _ in range(case["steps"]):
            ref.step()
        U = ref.moments(ref.f)
        out = [U[..., k].contiguous() for k in range(ref.d + 2)]
        if case["watch"]:
            c2 = torch.tensor([sum(k * k for k in c) for c in ref.c], dtype=U.dtype, device=U.device)
            energy = 0.5 * (c2 @ ref.f.reshape(ref.q, -1)).sum() + 0.5 * ref.d * ref.cs2 * U[..., 0].numel()
            rho, u, T, M = U[..., 0], [U[..., 1 + k] for k in range(ref.d)], U[..., -1], ref.M
            bulk = (rho * T - 1.0)[M:-M, M:-M] * ref.cs2
            v = [rho.sum(), *[(rho * x).sum() for x in u], energy, (bulk * bulk).sum(), sum(x * x for x in u).max().sqrt()]
            out.append(np.array([float(x) for x in v] + [0.0]))
        return out
