"""Performance cases: the work that programs have the solver do, from the smallest calls to the
largest, through the package's public entry points.

A pass is what a program does with one initial state: load the fields, project them when they are
noisy initial data, advance some steps, read the fields back.  The grid (with its workspace,
rheology, forcing, walls and obstacle) is made once and kept, as a program keeps it between
solves.  ``exact`` is the same method written with plain torch operations in 64 bits.
"""
from __future__ import annotations

import math

import torch

import paper_1803_09563_amd as evp

# transform lengths of the periodic directions (x additionally has to be even: all are)
LENGTHS = (8, 10, 12, 16, 20, 24, 30, 32, 40, 48, 60, 64, 80, 96, 120, 128, 160, 192, 240, 256,
           320, 384, 480, 512)
MODELS = {"oldroyd_b": evp.OLDROYD_B, "fene_p": evp.FENE_P, "saramito": evp.SARAMITO,
          "neo_hookean": evp.NEO_HOOKEAN}
DT = 1e-3

# alpha, zeta, xi of the three Runge-Kutta substeps
RK_ALPHA = (4 / 15, 1 / 15, 1 / 6)
RK_ZETA = (8 / 15, 5 / 12, 3 / 4)
RK_XI = (0.0, -17 / 60, -5 / 12)


def _case(name, nx, ny, nz, steps, walls=False, precision="fp64", model="saramito", scheme="weno",
          rk3=False, kappa=0.0, solid=False, moving=False, batch=1, restart=False, freeze=False):
    c = dict(nx=nx, ny=ny, nz=nz, steps=steps, walls=walls, precision=precision, model=model,
             scheme=scheme, rk3=rk3, kappa=kappa, solid=solid, moving=moving, batch=batch,
             restart=restart, freeze=freeze)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the uncoupled shear test of one material on the smallest box: launches and latency only
        _case("shear_8", 8, 8, 8, 25, freeze=True),
        # a small single solve (the smoke workload): latency of a step's chain of kernels
        _case("taylor_green_32", 32, 32, 32, 25, model="oldroyd_b"),
        # a chunk of the parameter-sweep serving loop: a batch of small solves of mixed models
        _case("serving_16x48", 48, 48, 48, 25, precision="mixed", model="sweep", batch=16),
        # initial projection alone, on lengths that are no powers of two
        _case("project_240", 240, 120, 160, 0),
        # Couette-type channel on ragged sizes with the linear upwind scheme, diffusion switched on
        _case("couette_120", 120, 75, 80, 10, walls=True, model="oldroyd_b", scheme="houc",
              kappa=1e-3, moving=True, restart=True),
        # wall-normal resolution above 256 rows
        _case("tall_channel_400", 96, 400, 64, 10, walls=True, model="fene_p"),
        # flow past a fixed sphere, periodic box
        _case("sphere_96", 96, 96, 96, 10, model="neo_hookean", solid=True),
        # the 128^3 turbulence workload in both precisions
        _case("kolmogorov_128", 128, 128, 128, 20),
        _case("kolmogorov_128_mixed", 128, 128, 128, 20, precision="mixed"),
        # the viscoelastic channel in the mixed form
        _case("channel_256_mixed", 256, 128, 128, 20, walls=True, precision="mixed", model="fene_p"),
        # the same channel with the Runge-Kutta integrator
        _case("channel_256_rk3", 256, 128, 128, 5, walls=True, rk3=True),
        # the largest workload: the elastoviscoplastic channel
        _case("channel_512", 512, 256, 256, 10, walls=True),
    ]


def draw(rng):
    """One more case: a single solve, a batch or a projection, of 2^9 to 2^24.5 cells."""
    kind = rng.choice(("step", "step", "step", "step", "batch", "project"))
    walls = kind != "batch" and rng.random() < 0.5
    cells = 2.0 ** rng.uniform(9.0, 24.5 if kind != "batch" else 17.0)
    best = None
    for _ in range(200):
        nx, nz = rng.choice(LENGTHS), rng.choice(LENGTHS)
        if walls:
            ny = max(4, min(512, int(cells / (nx * nz)) + rng.choice((0, 0, 1, 3))))
        else:
            ny = rng.choice(LENGTHS)
        if kind == "batch":
            ny = nz = nx
        off = abs(math.log(nx * ny * nz / cells)) + 0.2 * math.log(max(nx, ny, nz) / min(nx, ny, nz))
        if best is None or off < best[0]:
            best = (off, nx, ny, nz)
    _, nx, ny, nz = best
    n = nx * ny * nz
    if kind == "project":
        return _case(None, nx, ny, nz, 0, walls=walls)
    batch = rng.randint(2, 32) if kind == "batch" else 1
    rk3 = kind == "step" and rng.random() < 0.2
    most = 33554432 * 10 * 0.4 / (n * batch * (3.5 if rk3 else 1.0))
    steps = max(2, min(25, int(most)))
    scheme = "houc" if rng.random() < 0.2 else "weno"
    precision = rng.choice(("fp64", "mixed"))
    model = "sweep" if kind == "batch" else rng.choice(("oldroyd_b", "fene_p", "saramito", "saramito",
                                                        "neo_hookean"))
    solid = kind == "step" and n <= 2 ** 22 and rng.random() < 0.2
    restart = not rk3 and rng.random() < 0.3
    kappa = 1e-3 if precision == "fp64" and rng.random() < 0.2 else 0.0
    freeze = kind == "step" and not rk3 and not solid and rng.random() < 0.1
    return _case(None, nx, ny, nz, steps, walls=walls, precision=precision, model=model,
                 scheme=scheme, rk3=rk3, kappa=kappa, solid=solid, moving=walls and rng.random() < 0.3,
                 batch=batch, restart=restart, freeze=freeze)


# ---------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------

def _box(c):
    """(lx, ly, lz): 4 pi x 2 x 2 pi between walls, a 2 pi cube otherwise."""
    return (4 * math.pi, 2.0, 2 * math.pi) if c["walls"] else (2 * math.pi,) * 3


def _materials(c, seed):
    """Rheology of every grid of the case (rho = 1): the sweep draws model, Wi, Bi and beta."""
    g = torch.Generator().manual_seed(int(seed) + 17)
    out = []
    for b in range(c["batch"]):
        if c["model"] == "sweep":
            model = (evp.OLDROYD_B, evp.FENE_P, evp.SARAMITO)[(b + int(seed)) % 3]
            r = torch.rand(3, generator=g, dtype=torch.float64).tolist()
            wi, bi, beta, re = 0.1 + 9.9 * r[0], r[1], 0.1 + 0.8 * r[2], 1000.0
        else:
            model = MODELS[c["model"]]
            wi, bi, beta, re = {evp.OLDROYD_B: (1.0, 0.0, 0.5, 1000.0), evp.FENE_P: (5.0, 0.0, 0.9, 2000.0),
                                evp.SARAMITO: (2.0, 0.2, 0.1, 5000.0),
                                evp.NEO_HOOKEAN: (1.0, 0.0, 0.5, 1000.0)}[model]
        out.append(dict(model=model, rho=1.0, mu_s=beta / re, mu_p=(1 - beta) / re, lam=wi,
                        tau_y=bi / re if model == evp.SARAMITO else 0.0, L2=900.0))
    return out


def _forcing(c):
    if c["walls"]:
        return (evp.FORCE_CONST_X, 2.0 / 5000.0, 0.0)
    return (evp.FORCE_SIN_X_OF_Y, 1.0, 4.0)


def _wall_velocity(c):
    return (-0.5, 0.5, 0.1, -0.1) if c["moving"] else (0.0, 0.0, 0.0, 0.0)


def _fields(c, seed, b):
    """u, v, w, B and (for a restart) the history of grid b: a mean profile with noise, and a
    positive-definite conformation tensor I + a a^T of smooth stretched patches with a little
    noise (more of it where the artificial diffusion is to act)."""
    dev = "cuda"
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    lx, ly, lz = _box(c)
    shape = (nz, ny, nx)
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) * 64 + b)
    f64 = dict(device=dev, dtype=torch.float64)
    noise = lambda amp: (torch.rand(shape, generator=g, **f64) * 2 - 1) * amp  # noqa: E731
    y0 = -0.5 * ly if c["walls"] else 0.0
    yc = y0 + (torch.arange(ny, **f64) + 0.5) * (ly / ny)
    prof = 1.0 - yc ** 2 if c["walls"] else torch.sin(4.0 * yc)
    amp = 0.05 if c["walls"] else 0.01
    u = prof[None, :, None] + noise(amp)
    v, w = noise(amp), noise(amp)
    if c["walls"]:
        v[:, -1, :] = 0.0
    x = (torch.arange(nx, **f64) + 0.5) / nx * (2 * math.pi)
    y = (torch.arange(ny, **f64) + 0.5) / ny * (2 * math.pi)
    z = (torch.arange(nz, **f64) + 0.5) / nz * (2 * math.pi)
    ph = torch.rand(3, 3, generator=g, **f64) * (2 * math.pi)
    a = [0.7 * torch.sin(x + ph[m, 0])[None, None, :] * torch.cos(y + ph[m, 1])[None, :, None]
         * torch.cos((m + 1) * z + ph[m, 2])[:, None, None] for m in range(3)]
    B = torch.empty((6,) + shape, **f64)
    for cc, (p, q) in enumerate(((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))):
        B[cc] = a[p] * a[q] + (1.0 if p == q else 0.0) + noise(0.4 if c["kappa"] > 0 else 0.01)
    hist = None
    if c["restart"]:
        hist = torch.empty((9,) + shape, **f64)
        for cc in range(9):
            hist[cc] = a[cc % 3] * 0.2 + noise(0.05)
        if c["walls"]:
            hist[7, :, -1, :] = 0.0
    return u, v, w, B, hist


def _solid(c):
    """Solid fractions of a sphere around the velocity points, smoothed over a cell."""
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    lx, ly, lz = _box(c)
    y0 = -0.5 * ly if c["walls"] else 0.0
    f64 = dict(device="cuda", dtype=torch.float64)
    r0, out = 0.3 * min(lx, ly, lz), []
    h = max(lx / nx, ly / ny, lz / nz)
    for sx, sy, sz in ((1.0, 0.5, 0.5), (0.5, 1.0, 0.5), (0.5, 0.5, 1.0)):
        x = (torch.arange(nx, **f64) + sx) * (lx / nx) - 0.5 * lx
        y = y0 + (torch.arange(ny, **f64) + sy) * (ly / ny) - (0.0 if c["walls"] else 0.5 * ly)
        z = (torch.arange(nz, **f64) + sz) * (lz / nz) - 0.5 * lz
        r = torch.sqrt(x[None, None, :] ** 2 + y[None, :, None] ** 2 + z[:, None, None] ** 2)
        out.append(((r0 - r) / h + 0.5).clamp(0.0, 1.0).contiguous())
    if c["walls"]:
        out[1][:, -1, :] = 0.0
    return out


def prepare(case, seed):
    c = case
    prec = evp.MIXED if c["precision"] == "mixed" else evp.FP64
    grids, fields = [], []
    for b, mat in enumerate(_materials(c, seed)):
        G = evp.Grid(c["nx"], c["ny"], c["nz"], *_box(c), walls=c["walls"], precision=prec)
        G.set_rheology(**mat)
        G.set_forcing(*_forcing(c))
        if c["moving"]:
            G.set_walls(*_wall_velocity(c))
        if c["scheme"] == "houc" or c["kappa"] > 0:
            G.set_transport(evp.HOUC5 if c["scheme"] == "houc" else evp.WENO5, c["kappa"])
        if c["rk3"]:
            G.set_integrator(evp.RK3)
        if c["solid"]:
            G.set_solid(_solid(c))
        grids.append(G)
        fields.append(_fields(c, seed, b))
    return dict(case=c, grids=grids, fields=fields)


def _names(c):
    """What a pass reads out.  The mixed form's pressure is left out: it is the potential of the
    32-bit momentum increment divided by dt, whose rounding it carries amplified by 1/dt (1e-4 of
    its size at dt = 1e-3), so a program keeps the state it restarts from, u, v, w and B."""
    if c["freeze"]:
        return ("B",)
    if not c["steps"]:
        return ("u", "v", "w", "p")
    return ("u", "v", "w", "B") if c["precision"] == "mixed" else ("u", "v", "w", "p", "B")


def _kept(c, fields):
    """A program that computes its stresses in 32 bits keeps its snapshots in 32 bits."""
    return {k: t.float() for k, t in fields.items()} if c["precision"] == "mixed" else fields


def _gather(grids):
    """The fields of one solve, or those of a sweep's solves in one array each."""
    if len(grids) == 1:
        return grids[0]
    return {k: torch.stack([g[k] for g in grids]) for k in grids[0]}


def run(state):
    c, grids = state["case"], state["grids"]
    for G, (u, v, w, B, hist) in zip(grids, state["fields"]):
        G.write_fields(u, v, w, B, hist)
        if hist is None and not c["freeze"]:
            G.project()
    flags = evp.FREEZE_VELOCITY if c["freeze"] else 0
    if c["steps"]:
        if len(grids) > 1:
            evp.step_batch(grids, DT, c["steps"], flags)
        else:
            grids[0].step(DT, c["steps"], flags)
    return _gather([_kept(c, G.read_fields(_names(c))) for G in grids])


# ---------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------

def work(case):
    """Load (9 fields in 64 bits, 9 more of a restart) and read out; per step or
    substep the state read and written once (velocities in 64 bits; B and the two histories in 64
    or 32), the pressure written, and the half spectrum handed on once between the two directions of
    the Poisson solve.  About 1500 operations a cell for the stencils and 5 log2 N a transform."""
    c = case
    n = c["nx"] * c["ny"] * c["nz"]
    t = 4 if c["precision"] == "mixed" else 8
    io = 72 + (72 if c["restart"] else 0)
    poisson = 24
    fft = 2 * 2.5 * math.log2(n)
    if not c["steps"]:
        return {"bytes": float(n * (24 + 72 + 32 + poisson)), "flops": n * (fft + 30.0)}
    sub = c["steps"] * (3 if c["rk3"] else 1)
    if c["freeze"]:
        per, ops, out = 24 + 4 * 6 * t, 1000.0, 48
    else:
        per, ops, out = 48 + 2 * 15 * t + 8 + poisson, 1500.0 + fft, 80 if t == 8 else 36
    if c["solid"]:
        per += 24
    first = poisson + 56 if not c["restart"] and not c["freeze"] else 0
    return {"bytes": float(c["batch"] * n * (io + first + sub * per + out)),
            "flops": float(c["batch"] * n * sub * ops)}


# ---------------------------------------------------------------------------------------------
# the same method in plain torch, 64 bits
# ---------------------------------------------------------------------------------------------

class _Plain:
    """One grid.  Centre fields [nz][ny][nx]; velocities on the +x, +y, +z faces."""

    def __init__(self, c, mat):
        self.c, self.m = c, mat
        self.n = (c["nx"], c["ny"], c["nz"])
        self.h = tuple(length / n for length, n in zip(_box(c), self.n))
        self.walls, self.wv = c["walls"], _wall_velocity(c)
        f64 = dict(device="cuda", dtype=torch.float64)
        yc = (-1.0 if self.walls else 0.0) + (torch.arange(self.n[1], **f64) + 0.5) * self.h[1]
        kind, amp, ky = _forcing(c)
        self.fx = (torch.full_like(yc, amp) if kind == evp.FORCE_CONST_X else amp * torch.sin(ky * yc))[None, :, None]
        ev = lambda n, h: -(4 / h ** 2) * torch.sin(math.pi * torch.arange(n, **f64) / n) ** 2  # noqa: E731
        nx, ny, nz = self.n
        ex, ez = ev(nx, self.h[0])[:nx // 2 + 1], ev(nz, self.h[2])
        if self.walls:
            # cosine modes of the Neumann rows
            m = torch.arange(ny, **f64)
            ey = -(4 / self.h[1] ** 2) * torch.sin(math.pi * m / (2 * ny)) ** 2
            self.C = torch.cos(math.pi * m[:, None] * (m[None, :] + 0.5) / ny) * math.sqrt(2.0 / ny)
            self.C[0] *= math.sqrt(0.5)
        else:
            ey = ev(ny, self.h[1])
        self.eig = ez[:, None, None] + ey[None, :, None] + ex[None, None, :]
        self.eig[0, 0, 0] = 1.0

    # neighbours: offsets in x and z wrap; y rows come from an array with ghost rows
    @staticmethod
    def sh(f, i=0, k=0):
        if i:
            f = torch.roll(f, -i, -1)
        return torch.roll(f, -k, -3) if k else f

    def pad(self, f, g, kind):
        """g ghost rows in y: 'b' linear extrapolation, 'u'/'w' reflection about the wall, 'v'."""
        if not self.walls:
            return torch.cat([f[..., -g:, :], f, f[..., :g, :]], -2)
        lo, hi = [], []
        for q in range(1, g + 1):
            if kind == "b":
                lo.insert(0, (1 + q) * f[..., :1, :] - q * f[..., 1:2, :])
                hi.append((1 + q) * f[..., -1:, :] - q * f[..., -2:-1, :])
            elif kind == "v":
                lo.insert(0, torch.zeros_like(f[..., :1, :]))
                hi.append(torch.zeros_like(f[..., :1, :]))
            else:
                b, t = (self.wv[0], self.wv[1]) if kind == "u" else (self.wv[2], self.wv[3])
                lo.insert(0, 2 * b - f[..., q - 1:q, :])
                hi.append(2 * t - f[..., f.shape[-2] - q:f.shape[-2] - q + 1, :])
        return torch.cat(lo + [f] + hi, -2)

    def rows(self, f, g, j):
        return f[..., g + j:g + j + self.n[1], :]

    @staticmethod
    def weno(v1, v2, v3, v4, v5):
        s1 = 13 / 12 * (v1 - 2 * v2 + v3) ** 2 + 0.25 * (v1 - 4 * v2 + 3 * v3) ** 2
        s2 = 13 / 12 * (v2 - 2 * v3 + v4) ** 2 + 0.25 * (v2 - v4) ** 2
        s3 = 13 / 12 * (v3 - 2 * v4 + v5) ** 2 + 0.25 * (3 * v3 - 4 * v4 + v5) ** 2
        a1, a2, a3 = 0.1 / (1e-6 + s1) ** 2, 0.6 / (1e-6 + s2) ** 2, 0.3 / (1e-6 + s3) ** 2
        q = (a1 * (v1 / 3 - 7 / 6 * v2 + 11 / 6 * v3) + a2 * (-v2 / 6 + 5 / 6 * v3 + v4 / 3)
             + a3 * (v3 / 3 + 5 / 6 * v4 - v5 / 6))
        return q / (a1 + a2 + a3)

    def upwind(self, f, h, vel):
        d = [(f[m + 1] - f[m]) / h for m in range(6)]
        pos = vel >= 0
        v = [torch.where(pos, d[m], d[5 - m]) for m in range(5)]
        if self.c["scheme"] == "houc":
            return (2 * v[0] - 13 * v[1] + 47 * v[2] + 27 * v[3] - 3 * v[4]) / 60
        return self.weno(*v)

    def stress(self, B):
        m = self.m
        G = m["mu_p"] / m["lam"]
        if m["model"] == evp.FENE_P:
            F, a = m["L2"] / (m["L2"] - (B[0] + B[3] + B[5])), m["L2"] / (m["L2"] - 3)
            t = G * F * B
        else:
            a, t = 1.0, G * B
        for q in (0, 3, 5):
            t[q] -= G * a
        return t

    def rt(self, u, v, w, B):
        """Right-hand side of the conformation tensor."""
        m, sh, rows, (dx, dy, dz) = self.m, self.sh, self.rows, self.h
        U, V, W = self.pad(u, 1, "u"), self.pad(v, 1, "v"), self.pad(w, 1, "w")
        um = lambda j: rows(U, 1, j) + sh(rows(U, 1, j), -1)  # noqa: E731
        vs, ws, wm = v + rows(V, 1, -1), w + sh(w, 0, -1), lambda j: rows(W, 1, j) + sh(rows(W, 1, j), 0, -1)
        L = [[(u - sh(u, -1)) / dx, (um(1) - um(-1)) / (4 * dy), (sh(um(0), 0, 1) - sh(um(0), 0, -1)) / (4 * dz)],
             [(sh(vs, 1) - sh(vs, -1)) / (4 * dx), (v - rows(V, 1, -1)) / dy, (sh(vs, 0, 1) - sh(vs, 0, -1)) / (4 * dz)],
             [(sh(ws, 1) - sh(ws, -1)) / (4 * dx), (wm(1) - wm(-1)) / (4 * dy), (w - sh(w, 0, -1)) / dz]]
        uc, vc, wc = 0.5 * um(0), 0.5 * vs, 0.5 * ws
        G = m["mu_p"] / m["lam"]
        if m["model"] == evp.FENE_P:
            F, a = m["L2"] / (m["L2"] - (B[0] + B[3] + B[5])), m["L2"] / (m["L2"] - 3)
        elif m["model"] == evp.NEO_HOOKEAN:
            F, a = 0.0, 0.0
        elif m["model"] == evp.SARAMITO and m["tau_y"] > 0:
            tr = (B[0] + B[3] + B[5] - 3) / 3
            n2 = 0.5 * ((B[0] - 1 - tr) ** 2 + (B[3] - 1 - tr) ** 2 + (B[5] - 1 - tr) ** 2) + B[1] ** 2 + B[2] ** 2 + B[4] ** 2
            nrm = G * torch.sqrt(n2)
            F = torch.where(nrm > m["tau_y"], 1 - m["tau_y"] / nrm, torch.zeros_like(nrm))
            a = F
        else:
            F, a = 1.0, 1.0
        on = None
        if self.c["kappa"] > 0:
            det = (B[0] * (B[3] * B[5] - B[4] ** 2) - B[1] * (B[1] * B[5] - B[4] * B[2]) + B[2] * (B[1] * B[4] - B[3] * B[2]))
            on = det < 0
            if m["model"] == evp.FENE_P:
                on = on | (B[0] + B[3] + B[5] >= 0.95 * m["L2"])
        ix = ((0, 1, 2), (1, 3, 4), (2, 4, 5))
        out = torch.empty_like(B)
        for cc, (p, q) in enumerate(((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))):
            b = B[cc]
            P = self.pad(b, 3, "b")
            r = ((a if p == q else 0.0) - F * b) / m["lam"]
            r = r - uc * self.upwind([sh(b, i) for i in range(-3, 4)], dx, uc)
            r = r - vc * self.upwind([rows(P, 3, j) for j in range(-3, 4)], dy, vc)
            r = r - wc * self.upwind([sh(b, 0, k) for k in range(-3, 4)], dz, wc)
            for t in range(3):
                r = r + L[p][t] * B[ix[t][q]] + B[ix[p][t]] * L[q][t]
            if on is not None:
                lap = ((sh(b, 1) - 2 * b + sh(b, -1)) / dx ** 2 + (rows(P, 3, 1) - 2 * b + rows(P, 3, -1)) / dy ** 2
                       + (sh(b, 0, 1) - 2 * b + sh(b, 0, -1)) / dz ** 2)
                r = r + torch.where(on, self.c["kappa"] * lap, torch.zeros_like(lap))
            out[cc] = r
        return out

    def div_tau(self, B):
        sh, rows, (dx, dy, dz) = self.sh, self.rows, self.h
        T = self.stress(self.pad(B, 1, "b"))
        t = lambda q, j=0: rows(T[q], 1, j)  # noqa: E731
        xy = 0.25 * (T[1][:, :-1] + T[1][:, 1:])           # between rows j and j+1 (ghost rows included)
        xy = xy + sh(xy, 1)
        yz = 0.25 * (T[4][:, :-1] + T[4][:, 1:])
        yz = yz + sh(yz, 0, 1)
        xz = 0.25 * (t(2) + sh(t(2), 0, 1))
        xz = xz + sh(xz, 1)
        hi, lo = lambda f: f[:, 1:], lambda f: f[:, :-1]  # noqa: E731
        fx = (sh(t(0), 1) - t(0)) / dx + (hi(xy) - lo(xy)) / dy + (xz - sh(xz, 0, -1)) / dz
        fy = (hi(xy) - sh(hi(xy), -1)) / dx + (t(3, 1) - t(3)) / dy + (hi(yz) - sh(hi(yz), 0, -1)) / dz
        fz = (xz - sh(xz, -1)) / dx + (hi(yz) - lo(yz)) / dy + (sh(t(5), 0, 1) - t(5)) / dz
        return self.top([fx, fy, fz])

    def top(self, f):
        if self.walls:
            f[1][:, -1, :] = 0.0
        return f

    def advection(self, u, v, w):
        sh, rows, (dx, dy, dz) = self.sh, self.rows, self.h
        U, V, W = self.pad(u, 1, "u"), self.pad(v, 1, "v"), self.pad(w, 1, "w")
        up, un, vm, vn, wn = lambda j: rows(U, 1, j), rows(U, 1, 1), rows(V, 1, -1), rows(V, 1, 1), rows(W, 1, 1)
        uu = (0.5 * (u + sh(u, 1))) ** 2
        uv_lo = 0.25 * (vm + sh(vm, 1)) * (up(-1) + u)
        uv = 0.25 * (v + sh(v, 1)) * (u + un)
        uw = 0.25 * (w + sh(w, 1)) * (u + sh(u, 0, 1))
        vv = (0.5 * (v + vn)) ** 2
        vv_lo = (0.5 * (vm + v)) ** 2
        vw = 0.25 * (w + wn) * (v + sh(v, 0, 1))
        vw_lo = 0.25 * (rows(W, 1, -1) + w) * (vm + sh(vm, 0, 1))
        ww = (0.5 * (w + sh(w, 0, 1))) ** 2
        a = [(uu - sh(uu, -1)) / dx + (uv - uv_lo) / dy + (uw - sh(uw, 0, -1)) / dz,
             (uv - sh(uv, -1)) / dx + (vv - vv_lo) / dy + (vw - sh(vw, 0, -1)) / dz,
             (uw - sh(uw, -1)) / dx + (vw - vw_lo) / dy + (ww - sh(ww, 0, -1)) / dz]
        lap = lambda f, F: ((sh(f, 1) - 2 * f + sh(f, -1)) / dx ** 2 + (rows(F, 1, 1) - 2 * f + rows(F, 1, -1)) / dy ** 2  # noqa: E731
                            + (sh(f, 0, 1) - 2 * f + sh(f, 0, -1)) / dz ** 2)
        ms = self.m["mu_s"]
        return self.top(a), self.top([ms * lap(u, U), ms * lap(v, V), ms * lap(w, W)])

    def poisson(self, r):
        if not self.walls:
            q = torch.fft.rfftn(r, dim=(0, 1, 2)) / self.eig
            q[0, 0, 0] = 0.0
            return torch.fft.irfftn(q, s=r.shape, dim=(0, 1, 2))
        nz, ny, nx = r.shape
        y = lambda M, f: torch.mm(M, f.transpose(0, 1).reshape(ny, -1)).reshape(ny, nz, nx).transpose(0, 1)  # noqa: E731
        q = torch.fft.rfftn(y(self.C, r), dim=(0, 2)) / self.eig
        q[0, 0, 0] = 0.0
        return y(self.C.t().contiguous(), torch.fft.irfftn(q, s=(nz, nx), dim=(0, 2))).contiguous()

    def project(self, u, v, w, dt):
        sh, (dx, dy, dz) = self.sh, self.h
        V = self.pad(v, 1, "v")
        div = (u - sh(u, -1)) / dx + (v - self.rows(V, 1, -1)) / dy + (w - sh(w, 0, -1)) / dz
        p = self.poisson(div / dt)
        py = torch.cat([p[:, 1:], p[:, -1:] if self.walls else p[:, :1]], 1)
        u, v, w = u - dt * (sh(p, 1) - p) / dx, v - dt * (py - p) / dy, w - dt * (sh(p, 0, 1) - p) / dz
        self.top([u, v, w])
        return u, v, w, p

    def force(self, f, scale):
        f[0] = f[0] + scale * self.fx
        return f


def _solve(c, mat, fields, alpha):
    P = _Plain(c, mat)
    u, v, w, B, hist = fields
    p = torch.zeros_like(u)
    if hist is None and not c["freeze"]:
        u, v, w, p = P.project(u, v, w, 1.0)
    solid = (lambda f: [(1 - a) * x for a, x in zip(alpha, f)]) if alpha else (lambda f: f)
    rt0, ru0 = (hist[:6], [hist[6], hist[7], hist[8]]) if hist is not None else (None, None)
    for _ in range(c["steps"]):
        if c["rk3"]:
            rt0 = a0 = None
            for al, ze, xi in zip(RK_ALPHA, RK_ZETA, RK_XI):
                rt = P.rt(u, v, w, B)
                a, visc = P.advection(u, v, w)
                t0 = P.div_tau(B)
                B = B + DT * (ze * rt + (xi * rt0 if xi else 0.0))
                t1 = P.div_tau(B)
                rhs = P.force([-ze * x - (xi * y if xi else 0.0) + 2 * al * m + al * (s + t) for x, y, m, s, t in
                               zip(a, a0 or a, visc, t0, t1)], 2 * al)
                star = solid([f + DT * r for f, r in zip((u, v, w), rhs)])
                P.top(star)
                u, v, w, p = P.project(*star, 2 * al * DT)
                rt0, a0 = rt, a
            continue
        rt = P.rt(u, v, w, B)
        if not c["freeze"]:
            a, visc = P.advection(u, v, w)
            ru = P.force([-x + m + t for x, m, t in zip(a, visc, P.div_tau(B))], 1.0)
        B = B + DT * (rt if rt0 is None else 1.5 * rt - 0.5 * rt0)
        rt0 = rt
        if not c["freeze"]:
            star = [f + DT * (r if ru0 is None else 1.5 * r - 0.5 * r0) for f, r, r0 in zip((u, v, w), ru, ru0 or ru)]
            u, v, w, p = P.project(*solid(P.top(star)), DT)
            ru0 = ru
    return {"u": u, "v": v, "w": w, "p": p, "B": B}


def exact(case, seed):
    c = case
    alpha = _solid(c) if c["solid"] else None
    out = []
    for b, mat in enumerate(_materials(c, seed)):
        r = _solve(c, mat, _fields(c, seed, b), alpha)
        out.append({k: r[k] for k in _names(c)})
    return _gather(out)
