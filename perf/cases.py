"""Workloads of the particle-in-cell library whose speed is watched, each through its public entry points.

A case is a dict of plain values; `prepare` makes its inputs from a seed and the contexts, buffers and initial
fields that a program keeps; `run` is one pass; `work` is what a pass cannot do without; `exact` is what a pass
returns in plain torch in 64 bits. Kinds of case:

  steps   `Context.step`: a call of several electrostatic steps, as a time loop makes between two outputs. The
          fields, the energies and the bucket table come back, and with `snapshot` the particles too, in an order
          of their own (by cell, offset and velocity): the order inside a bucket is the library's. Ordering the
          particles of a large plasma would cost more than its steps, so there what depends on every one of them
          comes back alone: the fields of their charge at every node, their energies, the bucket table.
  em      `Context.em_step`: the same for the electromagnetic step.
  batch   `Batch.step`: an ensemble of small plasmas advanced together.
  grad    `FieldEnergyRun.forward` and `.backward`: a run's field energy and its gradient.
  setup   what starts every run: import of the physical state, sort, deposit, field, backward half push.
"""
import math

import torch

from paper_2608_15249_amd import workloads as W
from paper_2608_15249_amd.adjoint import FieldEnergyRun
from paper_2608_15249_amd.apic import Batch, Context, Particles

TWO_PI = 2.0 * math.pi


def _case(name, kind, dim, vdim, cells, n, dt, steps, *, length=None, prec="mixed", pusher="boris", c=0.0, bz=0.0,
          drift=0.0, spread=1.0, mode=0, delta=0.0, walls=False, snapshot=False, replicas=0, stride=0):
    nx, ny, nz = cells
    d = dict(kind=kind, dim=dim, vdim=vdim, nx=nx, ny=ny, nz=nz, n=n, dt=dt, steps=steps, prec=prec, pusher=pusher,
             c=c, bz=bz, length=length or float(nx), drift=drift, spread=spread, mode=mode, delta=delta, walls=walls,
             snapshot=snapshot, replicas=replicas, stride=stride)
    if name:
        d["name"] = name
    return d


def listed():
    return [
        # the smallest plasma a user runs: the 1D two-stream instability, where launches and latency count
        _case("two_stream_1d", "steps", 1, 1, (64, 1, 1), 16384, 0.1, 20, length=4 * math.pi, drift=1.0, spread=0.01,
              mode=1, delta=1e-3, snapshot=True),
        # the paper's own example: two beams in 64 x 64 cells, 2D3V
        _case("paper_two_stream", "steps", 2, 3, (64, 64, 1), 524288, 0.05, 40, drift=3.0, spread=1.0, mode=2,
              delta=0.005, snapshot=True),
        # sides that are not powers of two and a particle count that is no multiple of anything, in FP64
        _case("ragged_2d_fp64", "steps", 2, 2, (300, 182, 1), 1000003, 0.1, 20, prec="fp64", snapshot=True),
        # the non-periodic field solve between absorbing walls
        _case("walls_2d", "steps", 2, 2, (256, 256, 1), 4194304, 0.1, 20, walls=True),
        # the thermal plasma in full precision, ordinary size
        _case("thermal_2d_fp64", "steps", 2, 2, (512, 512, 1), 16777216, 0.1, 20, prec="fp64"),
        # the headline: a magnetized 2D3V plasma, the largest single run
        _case("magnetized_2d3v", "steps", 2, 3, (1024, 1024, 1), 33554432, 0.05, 20, bz=2.0, mode=16, delta=0.01),
        # the relativistic velocity advance on half that grid
        _case("relativistic_2d3v", "steps", 2, 3, (512, 512, 1), 8388608, 0.05, 20, pusher="hc", c=8.0, bz=2.0,
              mode=8, delta=0.01),
        # three dimensions
        _case("thermal_3d", "steps", 3, 3, (128, 128, 128), 16777216, 0.1, 20),
        # the electromagnetic step
        _case("em_2d3v", "em", 2, 3, (512, 512, 1), 8388608, 0.05, 20, c=10.0, bz=2.0, mode=8, delta=0.01),
        # the ensemble of uneven 1D plasmas
        _case("landau_batch", "batch", 1, 1, (0, 1, 1), 0, 0.1, 20, length=4 * math.pi, mode=1, replicas=256),
        # the gradient of a run: forward with checkpoints and the reverse sweep
        _case("gradient_2d", "grad", 2, 2, (256, 256, 1), 1048576, 0.1, 40, length=4 * math.pi, drift=1.0, spread=0.05,
              mode=1, delta=1e-3, stride=20),
        # the start of a run from particles in no order
        _case("setup_2d", "setup", 2, 2, (512, 512, 1), 16777216, 0.1, 1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["steps", "steps", "steps", "steps", "em", "batch", "grad", "setup"])
    prec = rng.choice(["mixed", "mixed", "fp64"])
    if kind == "batch":
        return _case(None, kind, 1, 1, (0, 1, 1), 0, 0.1, rng.randint(5, 20), length=4 * math.pi, mode=1,
                     replicas=_log(rng, 8, 200))
    dim = 2 if kind == "em" else rng.choice([1, 2, 2, 2, 3] if kind in ("steps", "setup") else [1, 2, 2, 3])
    vdim = {1: 1, 2: 3 if kind == "em" else rng.choice([2, 3]), 3: 3}[dim]
    most = {"steps": 1.6e7, "em": 8e6, "grad": 1e6, "setup": 1.6e7}[kind]
    n = _log(rng, 16384, most if dim > 1 else min(most, 2e6))
    per = rng.uniform(6, 64) if dim > 1 else rng.uniform(100, 400)   # particles per cell, about
    side = (n / per) ** (1.0 / dim)
    cells = [max(8, min({1: 1024, 2: 1024, 3: 128}[dim], int(round(side * rng.uniform(0.8, 1.25))))) if k < dim else 1
             for k in range(3)]
    if rng.random() < 0.5:   # half of them powers of two, the others as they come
        cells = [1 << int(round(math.log2(s))) if s > 1 else 1 for s in cells]
    walls = kind == "steps" and dim == 2 and rng.random() < 0.2
    pusher = "hc" if vdim == 3 and rng.random() < 0.3 else "boris"
    bz = rng.choice([0.0, 1.0, 2.0]) if vdim >= 2 else 0.0
    steps = {"steps": rng.randint(8, 20), "em": rng.randint(8, 20), "grad": rng.randint(8, 40), "setup": 1}[kind]
    return _case(None, kind, dim, vdim, tuple(cells), n, 0.05 if vdim == 3 else 0.1, steps, prec=prec, pusher=pusher,
                 c=10.0 if kind == "em" else (8.0 if pusher == "hc" else 0.0), bz=bz, mode=1, delta=0.01, walls=walls,
                 snapshot=kind == "steps" and n < 1000000, stride=rng.choice([5, 10, 20]) if kind == "grad" else 0)


# ---- inputs ----------------------------------------------------------------------------------------------------


def _box(c):
    d = c["length"] / c["nx"]
    return c["length"], d * c["ny"], d * c["nz"]


def _wrap(x, L):
    x = torch.remainder(x, L)
    return torch.where(x >= L, x - L, x)


def _plasma(c, seed):
    """Physical state in FP64: uniform positions with a displaced mode along x, drifting or thermal velocities."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = c["n"]
    pos = [torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * L for L in _box(c)[:c["dim"]]]
    vel = [torch.randn(n, generator=g, device="cuda", dtype=torch.float64) * c["spread"] for _ in range(c["vdim"])]
    if c["drift"]:
        vel[0][: n // 2] += c["drift"]
        vel[0][n // 2:] -= c["drift"]
    if c["mode"]:
        k = TWO_PI * c["mode"] / c["length"]
        pos[0] = _wrap(pos[0] + c["delta"] / k * torch.sin(k * pos[0]), c["length"])
    return pos, vel


def _replicas(c):
    return W.landau_batch(c["replicas"])


def _ensemble(c, seed):
    """Cells, offsets and velocities of all replicas, packed, and each particle's replica."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    reps = _replicas(c)
    of = torch.repeat_interleave(torch.arange(len(reps), device="cuda"),
                                 torch.tensor([r.n_particles for r in reps], device="cuda"))
    nx = torch.tensor([r.nx for r in reps], device="cuda", dtype=torch.float64)[of]
    delta = torch.tensor([r.delta0 for r in reps], device="cuda", dtype=torch.float64)[of]
    k = TWO_PI / c["length"]
    x = torch.rand(of.numel(), generator=g, device="cuda", dtype=torch.float64) * c["length"]
    x = _wrap(x + delta / k * torch.sin(k * x), c["length"])
    v = torch.randn(of.numel(), generator=g, device="cuda", dtype=torch.float64).float()
    at = x * nx / c["length"]
    cell = at.floor()
    off = (at - cell).float()
    cell = torch.where(off >= 1, cell + 1, cell)
    off = torch.where(off >= 1, torch.zeros_like(off), off)
    cell = torch.where(cell >= nx, cell - nx, cell)
    return cell.int(), off, v, of


def _split(x, d, n):
    """Cell and binary32 offset of a position, and the position they stand for in cells."""
    at = x / d
    cell = at.floor()
    off = (at - cell).float()
    cell = torch.where(off >= 1, cell + 1, cell)
    off = torch.where(off >= 1, torch.zeros_like(off), off)
    return torch.remainder(cell, n), off


def _context(c):
    lx, ly, lz = _box(c)
    return Context(dim=c["dim"], vdim=c["vdim"], nx=c["nx"], ny=c["ny"], nz=c["nz"], lx=lx, ly=ly, lz=lz, dt=c["dt"],
                   n=c["n"], bz=c["bz"], precision=c["prec"], pusher=c["pusher"], c_light=c["c"], walls=c["walls"],
                   model="em" if c["kind"] == "em" else "es")


def _import(c, ctx, p, pos, vel):
    if c["walls"]:   # the import of a physical state is for periodic plasmas
        if ctx.mixed:
            d = c["length"] / c["nx"]
            (ix, ox), (iy, oy) = (_split(x, d, m) for x, m in zip(pos, (c["nx"], c["ny"])))
            p.cell.copy_((iy.int() << 16) | ix.int())
            p.ox.copy_(ox)
            p.oy.copy_(oy)
        else:
            p.x.copy_(pos[0])
            p.y.copy_(pos[1])
        for dst, v in zip((p.vx, p.vy, p.vz), vel):
            dst.copy_(v)
        return
    ctx.import_state(p, pos[0], pos[1] if c["dim"] > 1 else None, *vel, z=pos[2] if c["dim"] == 3 else None)


def _start(s):
    """Sort, deposit, field of the initial charge and the backward half push."""
    ctx, p = s["ctx"], s["p"]
    ctx.sort_by_cell(p)
    ctx.deposit(p, s["rho"])
    ctx.field_solve(s["rho"], s["E"], s["E32"], s["we"])
    ctx.gather_push(p, s["E32"] if ctx.mixed else s["E"], dt_scale=-0.5, move=False)


def prepare(case, seed):
    c = case
    zeros = lambda n, t=torch.float64: torch.zeros(n, dtype=t, device="cuda")  # noqa: E731
    if c["kind"] == "batch":
        cell, off, v, of = _ensemble(c, seed)
        b = Batch([(r.nx, r.n_particles, c["length"]) for r in _replicas(c)], c["dt"])
        b.cell.copy_(cell)
        b.ox.copy_(off)
        b.vx.copy_(v)
        b.init()
        b.sync()
        return dict(case=c, batch=b, diag=zeros(c["steps"] * b.nrep * 4))
    pos, vel = _plasma(c, seed)
    if c["kind"] == "grad":
        lx, ly, lz = _box(c)
        run_ = FieldEnergyRun(dim=c["dim"], vdim=c["vdim"], nx=c["nx"], ny=c["ny"], nz=c["nz"], lx=lx, ly=ly, lz=lz,
                              dt=c["dt"], n=c["n"], nsteps=c["steps"], stride=c["stride"], bz=c["bz"],
                              precision=c["prec"], pusher=c["pusher"], c_light=c["c"])
        return dict(case=c, run=run_, pos=pos, vel=vel)
    ctx = _context(c)
    p = Particles(ctx)
    s = dict(case=c, ctx=ctx, p=p, diag=zeros(4 * c["steps"]))
    if c["kind"] == "em":
        s.update(F=zeros(6 * ctx.G), J=zeros(3 * ctx.G))
        _import(c, ctx, p, pos, vel)
        ctx.sort_by_cell(p)
        ctx.em_init_fields(p, s["F"])
        ctx.em_gather_push(p, s["F"], dt_scale=-0.5, move=False)
        ctx.sync()
        return s
    s.update(E=zeros(c["dim"] * ctx.G), E32=zeros(c["dim"] * ctx.G, torch.float32) if ctx.mixed else None,
             rho=zeros(ctx.G, torch.int64 if ctx.mixed else torch.float64), we=zeros(1))
    if c["kind"] == "setup":
        s.update(pos=pos, vel=vel)
        return s
    _import(c, ctx, p, pos, vel)
    _start(s)
    ctx.sync()
    return s


# ---- one pass --------------------------------------------------------------------------------------------------


def _arrays(p):
    return {k: getattr(p, k) for k in ("x", "y", "z", "cell", "ox", "oy", "oz", "vx", "vy", "vz")
            if getattr(p, k) is not None}


def _snapshot(p):
    """The particles by cell and offset (by position in FP64), equal ones by velocity."""
    by_v = torch.argsort(p.vx)
    key = p.x if p.cell is None else (p.cell.long() << 32) | p.ox.view(torch.int32).long()
    order = by_v[torch.argsort(key[by_v], stable=True)]
    return {k: a[order] for k, a in _arrays(p).items()}


def run(state):
    s = state
    c = s["case"]
    if c["kind"] == "batch":
        b = s["batch"]
        b.step(c["steps"], s["diag"])
        return dict(cell=b.cell, ox=b.ox, vx=b.vx, E=b.E, diag=s["diag"])
    if c["kind"] == "grad":
        r, pos, vel = s["run"], s["pos"], s["vel"]
        w = r.forward(pos[0], pos[1] if c["dim"] > 1 else None, *vel, *[None] * (3 - c["vdim"]),
                      z=pos[2] if c["dim"] == 3 else None)
        return dict(w=w, grad=r.backward())
    ctx, p = s["ctx"], s["p"]
    if c["kind"] == "em":
        ctx.em_step(p, s["F"], c["steps"], s["diag"], J=s["J"])
        return dict(F=s["F"], J=s["J"], diag=s["diag"], buckets=p.bucket_start)
    if c["kind"] == "setup":
        _import(c, ctx, p, s["pos"], s["vel"])
        _start(s)
        return dict(rho=s["rho"], E=s["E"], E32=s["E32"], we=s["we"], buckets=p.bucket_start, particles=_arrays(p))
    ctx.step(p, s["E"], s["E32"], c["steps"], s["diag"])
    out = dict(E=s["E"], E32=s["E32"], diag=s["diag"], buckets=p.bucket_start)
    if c["snapshot"]:
        out["particles"] = _snapshot(p)
    return out


def work(case):
    """Per step the particle state read and written once and the grid's charge and field once (the electromagnetic
    field and current); a gradient also walks back. The operations are those of gather, advance, move and deposit."""
    c = case
    if c["kind"] == "batch":
        n, g = sum(r.n_particles for r in _replicas(c)), sum(r.nx for r in _replicas(c))
        return dict(bytes=c["steps"] * (24.0 * n + 24.0 * g), flops=c["steps"] * 20.0 * n)
    dim, vdim, n = c["dim"], c["vdim"], c["n"]
    grid = c["nx"] * c["ny"] * c["nz"] * (2 if c["walls"] else 1)
    state = 4 * (1 + dim + vdim) if c["prec"] == "mixed" else 8 * (dim + vdim)
    flops = n * ((14 << dim) + 20.0)
    fft = 10.0 * grid * math.log2(max(grid, 2))
    if c["kind"] == "em":
        return dict(bytes=c["steps"] * (2.0 * state * n + 120.0 * grid), flops=c["steps"] * (n * 250.0 + 60.0 * grid))
    field = (8.0 + 8.0 * dim) * grid
    if c["kind"] == "setup":
        return dict(bytes=8.0 * (dim + vdim) * n + state * n + field, flops=flops + fft)
    passes = 2.0 if c["kind"] == "grad" else 1.0
    edge = 16.0 * (dim + vdim) * n if c["kind"] == "grad" else 0.0   # inputs read and gradients written
    return dict(bytes=edge + passes * c["steps"] * (2.0 * state * n + field), flops=passes * c["steps"] * (flops + fft))


# ---- the same in 64 bits ---------------------------------------------------------------------------------------


class _Ref:
    """The cycle in plain torch, FP64; positions in cells."""

    def __init__(self, c):
        self.c, self.dim, self.vdim = c, c["dim"], c["vdim"]
        self.d = c["length"] / c["nx"]
        self.real = [c["nx"], c["ny"], c["nz"]][:self.dim]
        self.cells = [2 * c["nx"] if c["walls"] else c["nx"], c["ny"], c["nz"]][:self.dim]   # walls: odd extension
        self.shape = tuple(reversed(self.cells))
        self.G = math.prod(self.cells)
        self.dV = self.d ** self.dim
        self.n0 = c["n"]
        self.Q = -math.prod(self.real) * self.dV / max(c["n"], 1)
        self.M = -self.Q
        self.dt, self.a = c["dt"], -0.5 * c["dt"]
        self.ic2 = 1.0 / c["c"] ** 2 if c["c"] and c["pusher"] == "hc" else 0.0

    def start(self, pos, vel):
        if self.c["prec"] == "mixed":
            both = [_split(x, self.d, n) for x, n in zip(pos, self.real)]
            return [cell + off.double() for cell, off in both], [v.float().double() for v in vel]
        return [x / self.d for x in pos], list(vel)

    def corners(self, g):
        """(node index, weight) of the 2^dim corners of each particle's cell."""
        base = [x.detach().floor() for x in g]
        out = []
        for k in range(1 << self.dim):
            idx, w, stride = 0, 1.0, 1
            for a in range(self.dim):
                hi = (k >> a) & 1
                i = torch.remainder(base[a].long() + hi, self.cells[a])
                f = g[a] - base[a]
                idx, w, stride = idx + i * stride, w * (f if hi else 1.0 - f), stride * self.cells[a]
            out.append((idx, w))
        return out

    def deposit(self, g):
        rho = torch.zeros(self.G, dtype=torch.float64, device="cuda")
        for idx, w in self.corners(g):
            rho = rho.index_add(0, idx, w)
        return 1.0 + rho * (self.Q / self.dV)

    def waves(self):
        k = []
        for a, n in enumerate(self.cells):
            m = torch.fft.fftfreq(n, device="cuda", dtype=torch.float64) * TWO_PI
            k.append(m.reshape([-1 if self.dim - 1 - b == a else 1 for b in range(self.dim)]))
        K2 = sum((2.0 / self.d * torch.sin(m / 2)) ** 2 for m in k)
        K2.reshape(-1)[0] = 1.0
        return k, K2

    def potential(self, rho):
        r = rho.reshape(self.shape)
        if self.c["walls"]:
            nx, odd = self.c["nx"], torch.zeros(self.shape, dtype=torch.float64, device="cuda")
            odd[:, 1:nx] = r[:, 1:nx]
            odd[:, nx + 1:] = -torch.flip(r[:, 1:nx], (1,))
            r = odd
        k, K2 = self.waves()
        f = torch.fft.fftn(r) / K2
        zero = torch.ones_like(K2)
        zero.reshape(-1)[0] = 0.0
        return k, f * zero

    def field(self, rho):
        k, phi = self.potential(rho)
        return [torch.fft.ifftn(phi * (-1j * torch.sin(m) / self.d)).real.reshape(-1) for m in k]

    def at(self, E, g):
        cs = self.corners(g)
        return [sum(w * e[i] for i, w in cs) for e in E]

    def advance(self, v, E, a):
        c, v = self.c, list(v)
        E = list(E) + [None] * (3 - len(E))
        m = [x if e is None else x + a * e for x, e in zip(v, E)]
        t = a * c["bz"]
        if c["pusher"] == "hc":
            g2 = 1.0 + sum(x * x for x in m) * self.ic2
            sig = g2 - t * t
            gp = torch.sqrt(0.5 * (sig + torch.sqrt(sig * sig + 4.0 * (t * t + (m[2] * t) ** 2 * self.ic2))))
            t = t / gp
        if c["bz"]:
            s = 2.0 * t / (1.0 + t * t)
            px, py = m[0] + m[1] * t, m[1] - m[0] * t
            m[0], m[1] = m[0] + py * s, m[1] - px * s
        return [x if e is None else x + a * e for x, e in zip(m, E)]

    def speed(self, v):
        if self.c["pusher"] != "hc":
            return v
        g = torch.sqrt(1.0 + sum(x * x for x in v) * self.ic2)
        return [x / g for x in v]

    def square(self, v):
        u2 = sum(x * x for x in v)
        return 2.0 * u2 / (torch.sqrt(1.0 + u2 * self.ic2) + 1.0) if self.c["pusher"] == "hc" else u2

    def energy(self, E):
        if self.c["walls"]:
            nx = self.c["nx"]
            w = torch.ones(nx + 1, dtype=torch.float64, device="cuda")
            w[0] = w[nx] = 0.5
            return 0.5 * self.dV * sum((w * e.reshape(self.shape)[:, :nx + 1] ** 2).sum() for e in E)
        return 0.5 * self.dV * sum((e * e).sum() for e in E)

    def move(self, g, v):
        g = [x + u * (self.dt / self.d) for x, u in zip(g, self.speed(v))]
        if self.c["walls"]:
            live = (g[0] >= 0) & (g[0] < self.c["nx"])
            g, v = [x[live] for x in g], [x[live] for x in v]
        return [_wrap(x, float(n)) for x, n in zip(g, self.cells)], v

    def step(self, g, v, E):
        old = self.square(v).sum()
        v = self.advance(v, self.at(E, g), self.a)
        ke, px = 0.25 * self.M * (old + self.square(v).sum()), self.M * v[0].sum()
        g, v = self.move(g, v)
        E = self.field(self.deposit(g))
        return g, v, E, torch.stack([self.Q * torch.tensor(float(g[0].numel()), device="cuda", dtype=torch.float64),
                                     self.energy(E), ke, px])


def _exact_em(c, pos, vel):
    r = _Ref(c)
    nx, ny, d, dt, c2 = c["nx"], c["ny"], r.d, c["dt"], c["c"] ** 2
    g, v = r.start(pos, vel)
    _, phi = r.potential(r.deposit(g))
    phi = torch.fft.ifftn(phi).real
    zero = torch.zeros_like(phi)
    F = [-(torch.roll(phi, -1, 1) - phi) / d, -(torch.roll(phi, -1, 0) - phi) / d, zero, zero, zero, zero + c["bz"]]
    half = [(1, 0), (0, 1), (0, 0), (0, 1), (1, 0), (1, 1)]   # components that sit half a cell up, by axis

    def at(F):
        return [r.at([f.reshape(-1)], [g[0] - 0.5 * h[0], g[1] - 0.5 * h[1]])[0] for f, h in zip(F, half)]

    def cross(p, q):
        return [p[1] * q[2] - p[2] * q[1], p[2] * q[0] - p[0] * q[2], p[0] * q[1] - p[1] * q[0]]

    def advance(v, f, a):
        m = [x + a * e for x, e in zip(v, f[:3])]
        t = [a * b for b in f[3:]]
        if c["pusher"] == "hc":
            t2 = sum(x * x for x in t)
            sig = 1.0 + sum(x * x for x in m) * r.ic2 - t2
            us = sum(x * y for x, y in zip(m, t))
            gp = torch.sqrt(0.5 * (sig + torch.sqrt(sig * sig + 4.0 * (t2 + us * us * r.ic2))))
            t = [x / gp for x in t]
        s = [2.0 * x / (1.0 + sum(y * y for y in t)) for x in t]
        q = [x + y for x, y in zip(m, cross(m, t))]
        return [x + y + a * e for x, y, e in zip(m, cross(q, s), f[:3])]

    def hat(x0, x1):
        """The four nodes from one below the old cell: index, old weight, change."""
        i0 = x0.floor()
        w = lambda x, k: (1.0 - (x - (i0 + k)).abs()).clamp_min(0.0)  # noqa: E731
        return i0.long() - 1, [w(x0, k) for k in (-1, 0, 1, 2)], [w(x1, k) - w(x0, k) for k in (-1, 0, 1, 2)]

    v = advance(v, at(F), -0.5 * r.a)
    diag = []
    for _ in range(c["steps"]):
        old = r.square(v).sum()
        v = advance(v, at(F), r.a)
        ke, px = 0.25 * r.M * (old + r.square(v).sum()), r.M * v[0].sum()
        u = r.speed(v)
        new = [x + w * (dt / d) for x, w in zip(g, u)]
        (ix, sx, dx), (iy, sy, dy) = hat(g[0], new[0]), hat(g[1], new[1])
        J = [torch.zeros(nx * ny, dtype=torch.float64, device="cuda") for _ in range(3)]
        sumx = [torch.zeros_like(ix, dtype=torch.float64) for _ in range(4)]
        for l in range(4):
            sumy = torch.zeros_like(sumx[0])
            for k in range(4):
                node = torch.remainder(iy + k, ny) * nx + torch.remainder(ix + l, nx)   # column l, row k
                sumy = sumy + dy[k] * (sx[l] + 0.5 * dx[l])
                sumx[k] = sumx[k] + dx[l] * (sy[k] + 0.5 * dy[k])
                J[0].index_add_(0, node, sumx[k] * (-r.Q / (d * dt)))
                J[1].index_add_(0, node, sumy * (-r.Q / (d * dt)))
                J[2].index_add_(0, node, u[2] * (r.Q / r.dV) * (sx[l] * sy[k] + 0.5 * (dx[l] * sy[k] + sx[l] * dy[k])
                                                               + dx[l] * dy[k] / 3.0))
        J = [j.reshape(ny, nx) for j in J]
        g = [_wrap(x, float(n)) for x, n in zip(new, (nx, ny))]
        up, dn = lambda f, ax: (torch.roll(f, -1, ax) - f) / d, lambda f, ax: (f - torch.roll(f, 1, ax)) / d  # noqa: E731

        def faraday(F):
            e = F[:3]
            return e + [F[3] - 0.5 * dt * up(e[2], 0), F[4] + 0.5 * dt * up(e[2], 1),
                        F[5] - 0.5 * dt * (up(e[1], 1) - up(e[0], 0))]

        F = faraday(F)
        b = F[3:]
        curl = [dn(b[2], 0), -dn(b[2], 1), dn(b[1], 1) - dn(b[0], 0)]
        F = faraday([e + dt * (c2 * q - j) for e, q, j in zip(F[:3], curl, J)] + b)
        wb = 0.5 * c2 * r.dV * ((F[3] ** 2).sum() + (F[4] ** 2).sum() + ((F[5] - c["bz"]) ** 2).sum())
        diag.append(torch.stack([wb, r.energy(F[:3]), ke, px]))
    return dict(F=torch.stack(F).reshape(-1), J=torch.stack(J).reshape(-1), diag=torch.cat(diag), buckets=None)


def _exact_batch(c, seed):
    cell, off, v, of = _ensemble(c, seed)
    reps, dt = _replicas(c), c["dt"]
    nx = torch.tensor([r.nx for r in reps], device="cuda")
    first = torch.cumsum(nx, 0) - nx
    total = int(nx.sum())
    d = torch.tensor([c["length"] / r.nx for r in reps], device="cuda", dtype=torch.float64)
    q = torch.tensor([-c["length"] / r.n_particles for r in reps], device="cuda", dtype=torch.float64)
    node_rep = torch.repeat_interleave(torch.arange(len(reps), device="cuda"), nx)
    nxp, base, shift = nx[of], first[of], (dt / d)[of]
    g, v = cell.double() + off.double(), v.double()
    size = nxp.double()

    def corners(g):
        i = g.floor()
        f = g - i
        i = i.long()
        return base + i, base + torch.where(i + 1 >= nxp, torch.zeros_like(i), i + 1), f

    def field(g):
        lo, hi, f = corners(g)
        rho = torch.zeros(total, dtype=torch.float64, device="cuda").index_add(0, lo, 1.0 - f).index_add(0, hi, f)
        rho = 1.0 + rho * (q / d)[node_rep]
        out = []
        for k, r in enumerate(reps):
            m = torch.fft.rfftfreq(r.nx, device="cuda", dtype=torch.float64) * TWO_PI
            h = c["length"] / r.nx
            K2 = (2.0 / h * torch.sin(m / 2)) ** 2
            K2[0] = 1.0
            s = -1j * torch.sin(m) / h / K2
            s[0] = 0.0
            a = int(first[k])
            out.append(torch.fft.irfft(torch.fft.rfft(rho[a:a + r.nx]) * s, n=r.nx))
        return torch.cat(out)

    def at(E, g):
        lo, hi, f = corners(g)
        return (1.0 - f) * E[lo] + f * E[hi]

    per = lambda x, of, w: torch.zeros(len(reps), dtype=torch.float64, device="cuda").index_add(0, of, x) * w  # noqa: E731
    count = torch.tensor([r.n_particles for r in reps], device="cuda")
    end = torch.cumsum(count, 0)

    def total_of(x):
        s = torch.cumsum(x, 0)[end - 1]
        return torch.diff(s, prepend=s.new_zeros(1))

    E = field(g)
    v = v + 0.5 * dt * at(E, g)
    diag = []
    for _ in range(c["steps"]):
        old = v * v
        v = v - dt * at(E, g)
        ke, px = -0.25 * q * total_of(old + v * v), -q * total_of(v)
        g = torch.remainder(g + v * shift, size)
        g = torch.where(g >= size, g - size, g)
        E = field(g)
        diag.append(torch.stack([q * count, 0.5 * d * per(E * E, node_rep, 1.0), ke, px], 1).reshape(-1))
    return dict(cell=None, ox=None, vx=v, E=E, diag=torch.cat(diag))


def exact(case, seed):
    c = case
    if c["kind"] == "batch":
        return _exact_batch(c, seed)
    pos, vel = _plasma(c, seed)
    if c["kind"] == "em":
        return _exact_em(c, pos, vel)
    r = _Ref(c)
    g, v = r.start(pos, vel)
    if c["kind"] == "grad":
        if c["n"] * c["steps"] * (16 << c["dim"]) * 8 * 2 > 100e9:
            return None   # the graph would not fit
        x = [(a * r.d).requires_grad_() for a in g]
        v0 = [a.requires_grad_() for a in v]
        g = [a / r.d for a in x]
        E = r.field(r.deposit(g))
        v = r.advance(v0, r.at(E, g), -0.5 * r.a)
        for _ in range(c["steps"]):
            v = r.advance(v, r.at(E, g), r.a)
            g, v = r.move(g, v)
            E = r.field(r.deposit(g))
        w = r.energy(E)
        grads = torch.autograd.grad(w, x + v0)
        dim, vdim = c["dim"], c["vdim"]
        gx, gv = list(grads[:dim]) + [None] * (3 - dim), list(grads[dim:]) + [None] * (3 - vdim)
        return dict(w=w.detach().reshape(1), grad=[gx[0], gx[1], gv[0], gv[1], gv[2], gx[2]])
    E = r.field(r.deposit(g))
    if c["kind"] == "setup":
        all_E = torch.cat(E)
        return dict(rho=None if c["prec"] == "mixed" else r.deposit(g), E=all_E,
                    E32=all_E if c["prec"] == "mixed" else None, we=r.energy(E).reshape(1), buckets=None,
                    particles=None)
    v = r.advance(v, r.at(E, g), -0.5 * r.a)
    diag = []
    for _ in range(c["steps"]):
        g, v, E, row = r.step(g, v, E)
        diag.append(row)
    all_E = torch.cat(E)
    return dict(E=all_E, E32=all_E if c["prec"] == "mixed" else None, diag=torch.cat(diag), buckets=None)
