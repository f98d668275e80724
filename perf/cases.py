"""The work that programs have this solver do, as measurable cases.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges,
``prepare`` builds what a program holds before the call (inputs on the device,
a solver context), ``run`` is one pass through the public entry points, ``work``
the bytes and operations that pass cannot do without, and ``exact`` the same
results from plain torch transforms in 64 bits.

Kinds of case
-------------
solve     one whole solve: set the initial state, advance ``steps`` time steps
          (``rk_step`` or graph replay), read the state back.  Every pass starts
          from the same initial fields, as a served request or a parameter
          sweep does.
serve     the request loop over several solves of mixed shapes, host arrays in
          and out.
rhs       the advective term of given physical fields.
project   the pressure projection of a given physical field.
derivative, extend   the wall-normal FC-Gram operators on a batch of lines.
"""
import math
import os

import numpy as np
import torch

import paper_2002_01392_amd as fcns

DEV = "cuda:0" if torch.cuda.is_available() else "cpu"
TABLES = os.path.join(os.path.dirname(os.path.abspath(fcns.__file__)), "tables")


# ---------------------------------------------------------------- the cases
def _solve(flow, nx, ny, nz, steps, C=31, d=5, order=2, precision="fp64", how="step",
           tuned=False, pressure=False, stats=False, re=1000.0, dt=0.0):
    c = dict(kind="solve", flow=flow, nx=nx, ny=ny, nz=nz, C=C, d=d, re=re, steps=steps,
             order=order, precision=precision, how=how, tuned=tuned, pressure=pressure,
             stats=stats, dt=dt)
    if dt == 0.0:
        c["dt"] = _stable_dt(c)
    return c


def listed():
    return [
        # the smallest grid: launches and latency (the paper's laminar channel set-up,
        # N' = 58 = 2 x 29)
        dict(_solve("channel", 32, 32, 33, 10, C=25, dt=1e-3), name="channel_32"),
        # a small convection solve stepped by graph replay
        dict(_solve("rb", 64, 64, 65, 20, how="graph", re=1e6), name="rb_64_graph"),
        # the request loop of a parameter sweep: six solves of four sizes
        dict(kind="serve", sides="32,32,64,64,96,128", steps=20, name="serve_mix"),
        # one large request of that sweep, default launch choices
        dict(_solve("rb", 192, 192, 193, 20, re=1e7), name="rb_192"),
        # the headline convection grid, launch choices tuned as a long run does
        dict(_solve("rb", 512, 512, 257, 4, tuned=True, re=1e8, dt=1e-3), name="rb_512"),
        # the turbulent channel with pressure and flow statistics (N' = 282 = 2 x 3 x 47)
        dict(_solve("loglaw", 256, 256, 257, 5, C=25, tuned=True, pressure=True, stats=True,
                    dt=2e-4), name="channel_256"),
        # the same grid in mixed precision
        dict(_solve("loglaw", 256, 256, 257, 5, C=25, tuned=True, precision="mixed", dt=2e-4),
             name="channel_256_mixed"),
        # a box of no particular size, three stages, default choices (N' = 106 = 2 x 53)
        dict(_solve("rb", 120, 84, 81, 10, C=25, order=3, re=1e6), name="rb_ragged"),
        # the operators on their own
        dict(kind="rhs", nx=256, ny=192, nz=129, C=31, d=5, theta=True, filtered=True,
             name="rhs_filtered"),
        dict(kind="project", nx=160, ny=160, nz=161, C=25, d=5, name="project_160"),
        dict(kind="derivative", lines=65537, nz=257, C=31, d=5, order=1, name="derivative_257"),
        dict(kind="extend", lines=50001, nz=193, C=25, d=5, name="extend_193"),
    ]


def _loguni(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _even(rng, lo, hi):
    # lengths in use: powers of two with a small factor, and now and then any even number
    if rng.random() < 0.25:
        return 2 * int(round(_loguni(rng, lo, hi) / 2))
    ok = [m << k for m in (1, 3, 5, 7, 9, 15) for k in range(1, 10) if lo <= m << k <= hi]
    return ok[min(range(len(ok)), key=lambda i, t=_loguni(rng, lo, hi): abs(ok[i] - t))]


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "serve", "rhs", "project", "derivative",
                       "extend"])
    C, d = rng.choice([(31, 5), (31, 5), (25, 5), (15, 5), (33, 7)])
    if kind in ("derivative", "extend"):
        nz = 2 * int(round(_loguni(rng, 16, 128))) + 1
        c = dict(kind=kind, lines=int(_loguni(rng, 100, 100000)), nz=nz, C=C, d=d)
        if kind == "derivative":
            c["order"] = rng.choice([1, 2])
        return c
    if kind == "serve":
        sides = [rng.choice([32, 64, 96, 128]) for _ in range(rng.randint(2, 6))]
        return dict(kind=kind, sides=",".join(map(str, sides)), steps=rng.choice([5, 10, 20]))
    while True:
        nx, ny = _even(rng, 16, 320), _even(rng, 16, 320)
        nz = rng.choice([2 * int(round(_loguni(rng, 16, 128))) + 1, 33, 65, 97, 129, 193, 257])
        if nx * ny * nz <= 5e6:
            break
    if kind == "rhs":
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, C=C, d=d, theta=rng.random() < 0.5,
                    filtered=rng.random() < 0.5)
    if kind == "project":
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, C=C, d=d)
    precision = rng.choice(["fp64", "fp64", "fp64", "mixed"])
    flow = rng.choice(["rb", "channel"])
    re = _loguni(rng, 1e4, 1e8) if flow == "rb" else _loguni(rng, 500, 5000)
    return _solve(flow, nx, ny, nz, rng.choice([3, 5, 8]), C=C, d=d,
                  order=rng.choice([2, 2, 2, 1, 3]), precision=precision,
                  how=rng.choice(["step", "step", "graph"]), tuned=rng.random() < 0.3,
                  pressure=precision == "fp64" and ny >= 64 and rng.random() < 0.3,
                  stats=rng.random() < 0.2, re=float("%.4g" % re))


# ---------------------------------------------------------------- problems and inputs
def _physics(c):
    """Box, viscosity and forcing of a flow (re: Re of the channel, Ra of convection)."""
    flow = c.get("flow", "channel")
    if flow == "rb":                       # convection, box 2 x 2 x 1, Pr = 1
        nu = math.sqrt(1.0 / c["re"])
        return dict(lx=2.0, ly=2.0, lz=1.0, nu=nu, kappa=nu, gamma=1.0, boussinesq=True,
                    forcing_x=0.0)
    box = dict(lx=4 * math.pi, ly=2 * math.pi, lz=2.0, kappa=0.0, gamma=0.0, boussinesq=False)
    if flow == "loglaw":                   # turbulent channel at Re_tau = 180
        return dict(box, nu=1.0 / 180.0, forcing_x=1.0)
    nu = 2.0 * (2.0 / 3.0) / c.get("re", 1000.0)
    if c.get("theta"):
        box = dict(box, kappa=nu, gamma=1.0, boussinesq=True)
    return dict(box, nu=nu, forcing_x=8.0 * nu / 4.0)


def _stable_dt(c):
    p = _physics(c)
    k2 = sum((math.pi * n / l) ** 2
             for n, l in ((c["nx"], p["lx"]), (c["ny"], p["ly"]), (c["nz"] - 1, p["lz"])))
    return min(1e-3, 1.0 / (p["nu"] * k2))


def _harmonics(n, length, kmax):
    """cos and sin of the modes 0..kmax on n points, and their derivatives."""
    k = torch.arange(0, kmax + 1, dtype=torch.float64, device=DEV) * (2 * math.pi / length)
    x = torch.arange(n, dtype=torch.float64, device=DEV) * (length / n)
    ph = x[:, None] * k[None]
    return (torch.cat([torch.cos(ph), torch.sin(ph)], 1),
            torch.cat([-k * torch.sin(ph), k * torch.cos(ph)], 1))


def _field(a, bz, by, bx):
    """sum_mpq a[m, p, q] bz[z, m] by[y, p] bx[x, q] as [z][y][x]."""
    m, b, _ = a.shape
    t = (bz @ a.reshape(m, -1)).reshape(bz.shape[0], b, b)
    t = torch.matmul(by, t)
    return (t.reshape(-1, b) @ bx.t().contiguous()).reshape(bz.shape[0], by.shape[0], bx.shape[0])


def _wall_modes(nz, lz, mmax):
    z = torch.arange(nz, dtype=torch.float64, device=DEV) * (lz / (nz - 1))
    k = torch.arange(1, mmax + 1, dtype=torch.float64, device=DEV) * (math.pi / lz)
    h2 = (lz / 2) ** 4
    g, gp = (z * (lz - z)) ** 2 / h2, 2 * z * (lz - z) * (lz - 2 * z) / h2
    s, c = torch.sin(z[:, None] * k), torch.cos(z[:, None] * k)
    return z, s, s * g[:, None], k * c * g[:, None] + s * gp[:, None]


def _noise(gen, nx, ny, nz, lx, ly, lz, rms, kmax=4, mmax=4):
    """A solenoidal field vanishing at the walls (a curl), scaled to rms."""
    fx, dfx = _harmonics(nx, lx, kmax)
    fy, dfy = _harmonics(ny, ly, kmax)
    _, _, zm, dzm = _wall_modes(nz, lz, mmax)
    a = torch.randn(3, mmax, 2 * kmax + 2, 2 * kmax + 2, dtype=torch.float64, device=DEV,
                    generator=gen)
    v = torch.stack([_field(a[2], zm, dfy, fx) - _field(a[1], dzm, fy, fx),
                     _field(a[0], dzm, fy, fx) - _field(a[2], zm, fy, dfx),
                     _field(a[1], zm, fy, dfx) - _field(a[0], zm, dfy, fx)])
    return v * (rms / v.square().sum(0).mean().sqrt())


def _scalar(gen, nx, ny, nz, lx, ly, lz, rms, kmax=4, mmax=4):
    """A scalar vanishing at the walls, scaled to rms."""
    fx, _ = _harmonics(nx, lx, kmax)
    fy, _ = _harmonics(ny, ly, kmax)
    _, s, _, _ = _wall_modes(nz, lz, mmax)
    s[-1] = 0.0
    a = torch.randn(mmax, 2 * kmax + 2, 2 * kmax + 2, dtype=torch.float64, device=DEV,
                    generator=gen)
    f = _field(a, s, fy, fx)
    return f * (rms / f.square().mean().sqrt())


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _initial(c, seed):
    """(v, theta) of a solve: the flow's mean profile plus solenoidal noise."""
    p, g = _physics(c), _gen(seed)
    shape = (c["nx"], c["ny"], c["nz"], p["lx"], p["ly"], p["lz"])
    z = torch.arange(c["nz"], dtype=torch.float64, device=DEV) * (p["lz"] / (c["nz"] - 1))
    kmax = min(8, c["nx"] // 4, c["ny"] // 4) if c["nx"] >= 256 else 4
    if p["boussinesq"]:
        v = _noise(g, *shape, 1e-3, kmax)
        return v, _scalar(g, *shape, 1e-3, kmax)
    if c["flow"] == "loglaw":              # Reichardt's composite profile in wall units
        zp = z * (p["lz"] - z) / p["lz"] / p["nu"]
        u = torch.log1p(0.41 * zp) / 0.41 + 7.8 * (
            1.0 - torch.exp(-zp / 11.0) - (zp / 11.0) * torch.exp(-zp / 3.0))
        v = _noise(g, *shape, 0.1 * float(u.mean()), kmax)
    else:                                  # laminar profile, u_max = 1
        u = p["forcing_x"] * z * (p["lz"] - z) / (2.0 * p["nu"])
        v = _noise(g, *shape, 1e-3, kmax)
    v[0] += u[:, None, None]
    return v, None


def _rhs_input(c, seed):
    """A laminar profile with strong noise (and a scalar): fields with non-zero products."""
    p, g = _physics(c), _gen(seed)
    shape = (c["nx"], c["ny"], c["nz"], p["lx"], p["ly"], p["lz"])
    v = _noise(g, *shape, 0.2)
    z = torch.arange(c["nz"], dtype=torch.float64, device=DEV) * (p["lz"] / (c["nz"] - 1))
    v[0] += (z * (p["lz"] - z))[:, None, None]
    return v, (_scalar(g, *shape, 0.2) if c.get("theta") else None)


def _project_input(c, seed):
    """A solenoidal field plus c grad p of a smooth pressure: a stage's pressureless field."""
    p, g = _physics(c), _gen(seed)
    shape = (c["nx"], c["ny"], c["nz"], p["lx"], p["ly"], p["lz"])
    v = _noise(g, *shape, 0.2)
    for i in range(3):
        v[i] += _scalar(g, *shape, 0.02)
    return v


def _lines_input(c, seed):
    """Smooth lines that do not vanish at the ends: low harmonics plus a cubic."""
    g = _gen(seed)
    z = torch.linspace(0.0, 1.0, c["nz"], dtype=torch.float64, device=DEV)
    basis = torch.stack([z ** k for k in range(4)] + [torch.sin(3.7 * k * z + k)
                                                      for k in range(1, 6)])
    a = torch.randn(c["lines"], basis.shape[0], dtype=torch.float64, device=DEV, generator=g)
    return (a @ basis).contiguous()


def _serve_requests(c):
    """Solve cases of a sweep: convection and channel in turn, one per side."""
    out = []
    for i, side in enumerate(int(s) for s in c["sides"].split(",")):
        out.append(_solve("rb" if i % 2 else "channel", side, side, side + 1, c["steps"],
                          re=1e6 if i % 2 else 1000.0 + 300.0 * i))
    return out


# ---------------------------------------------------------------- prepare and run
def prepare(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind == "serve":
        srv = fcns.Server(max_active=8, max_bytes=32 << 30)
        reqs = []
        for i, r in enumerate(_serve_requests(c)):
            p = _physics(r)
            prob, tab = fcns.make_problem(r["nx"], r["ny"], r["nz"], d=r["d"], C=r["C"], **p)
            v, th = _initial(r, seed * 100 + i)
            reqs.append((prob, tab, v.cpu().numpy(), th.cpu().numpy() if th is not None else None,
                         r["dt"], r["steps"]))
        return dict(case=c, srv=srv, reqs=reqs)
    if kind in ("derivative", "extend"):
        s = fcns.Solver(8, 8, c["nz"], 1.0, 1.0, 1.0, 1e-3, d=c["d"], C=c["C"])
        return dict(case=c, solver=s, lines=_lines_input(c, seed))
    p = _physics(c)
    s = fcns.Solver(c["nx"], c["ny"], c["nz"], d=c["d"], C=c["C"],
                    keep_pressure=c.get("pressure", False), rk_order=c.get("order", 2),
                    precision=c.get("precision", "fp64"), **p)
    if kind == "project":
        return dict(case=c, solver=s, v=_project_input(c, seed))
    if kind == "rhs":
        v, th = _rhs_input(c, seed)
        return dict(case=c, solver=s, v=v, theta=th)
    v, th = _initial(c, seed)
    if c["tuned"]:
        s.set_state(v, th)
        s.autotune()
    return dict(case=c, solver=s, v=v, theta=th)


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "serve":
        srv = state["srv"]
        ids = [srv.submit(prob, v, th, dt, n) for prob, _, v, th, dt, n in state["reqs"]]
        while True:
            queued, active, _ = srv.poll()
            if queued + active == 0:
                break
        out = []
        for i in ids:
            v, th, info = srv.result(i)
            if info["status"] != 0:
                raise RuntimeError("a served request failed")
            out.append((v, th))
            srv.release(i)
        return out
    s = state["solver"]
    if kind == "extend":
        return s.fc_extend(state["lines"])
    if kind == "derivative":
        return s.fc_derivative(state["lines"], c["order"])
    if kind == "project":
        return s.pressure_project(state["v"], 1e-3)
    if kind == "rhs":
        return s.rhs_nonlinear(state["v"], state["theta"], filtered=c["filtered"])
    s.set_state(state["v"], state["theta"])
    (s.rk_graph if c["how"] == "graph" else s.rk_step)(c["dt"], c["steps"])
    out = list(s.get_state(pressure=c["pressure"]))
    if c["precision"] == "mixed":
        # a mixed-precision run keeps its fields as float32
        out = [None if x is None else x.float() for x in out]
    if c["stats"]:
        out.append(np.array(list(s.diagnostics().values())))
        out.extend(s.spectra(0, c["nz"] // 2))
    return out


# ---------------------------------------------------------------- work
def _fft_flops(n):
    return 5.0 * n * math.log2(n)


def _step_work(c):
    """One RK stage: the continued state read and written once, and the mixed-space fields
    and the nonlinear term crossing memory once each way between the wall-normal and the
    horizontal transforms (neither direction's lines fit on the chip together)."""
    nf = 4 if _physics(c)["boussinesq"] else 3
    nx, ny, nz, npr = c["nx"], c["ny"], c["nz"], c["nz"] + c["C"]
    pen = (nx // 2 + 1) * ny
    mixed = 8 if c["precision"] == "mixed" else 16
    by = nf * pen * (2 * 16 * npr + 4 * mixed * nz)
    fl = pen * (5 * nf + 1) * _fft_flops(npr)
    fl += nf * nz * (4 * (nx // 2 + 1) * _fft_flops(ny) + 5 * ny * _fft_flops(nx) / 2)
    return by, fl


def work(case):
    c = dict(case)
    kind = c["kind"]
    if kind == "serve":
        ws = [work(r) for r in _serve_requests(c)]
        return dict(bytes=sum(w["bytes"] for w in ws), flops=sum(w["flops"] for w in ws))
    nz, npr = c["nz"], c["nz"] + c["C"]
    if kind == "extend":
        return dict(bytes=8.0 * c["lines"] * (nz + npr), flops=4.0 * c["lines"] * c["C"] * c["d"])
    if kind == "derivative":
        return dict(bytes=16.0 * c["lines"] * nz,
                    flops=c["lines"] * (_fft_flops(npr) + 4.0 * c["C"] * c["d"]))
    nx, ny = c["nx"], c["ny"]
    pts, pen = nx * ny * nz, (nx // 2 + 1) * ny
    xy = nz * ((nx // 2 + 1) * _fft_flops(ny) + ny * _fft_flops(nx) / 2)
    if kind == "project":
        return dict(bytes=6 * 8.0 * pts + 12 * 16.0 * pen * nz,
                    flops=6 * xy + 7 * pen * _fft_flops(npr))
    if kind == "rhs":
        nf = 4 if c["theta"] else 3
        # into mixed space and back around the z transforms (twice when filtered)
        n = nf * (3 if c["filtered"] else 1)
        return dict(bytes=2 * nf * 8.0 * pts + n * 2 * 16.0 * pen * nz,
                    flops=6 * nf * xy + (3 + 2 * c["filtered"]) * nf * pen * _fft_flops(npr))
    by, fl = _step_work(c)
    nf = 4 if _physics(c)["boussinesq"] else 3
    n = c["steps"] * c["order"]
    return dict(bytes=n * by + 2 * nf * 8.0 * pts, flops=n * fl + 2 * nf * xy)


# ---------------------------------------------------------------- exact
def _modes(n):
    """Signed mode numbers in transform order, the even Nyquist one negative."""
    m = torch.arange(n)
    return torch.where(2 * m < n, m, m - n)


class _Plain:
    """The scheme from its formulas in plain torch transforms, 64 bits."""

    def __init__(self, nx, ny, nz, C, d, lx, ly, lz, nu, kappa=0.0, gamma=0.0,
                 boussinesq=False, forcing_x=0.0):
        self.__dict__.update(nx=nx, ny=ny, nz=nz, C=C, d=d, lz=lz, nu=nu, kappa=kappa,
                             gamma=gamma, boussinesq=boussinesq, forcing_x=forcing_x)
        t = torch.from_numpy(np.loadtxt(os.path.join(TABLES, f"fc_d{d}_C{C}.txt"))).to(DEV)
        self.m_r = t[d * d:].reshape(C, d) @ t[:d * d].reshape(d, d).t()
        self.n = n = nz + C
        self.dz = lz / (nz - 1)

        def waves(m, count, scale):
            m = m.to(DEV, torch.float64)
            k = m * scale
            return k, torch.where(2 * m.abs() == count, torch.zeros_like(k), k), m.abs() / count
        kx, ox, ex = waves(torch.arange(nx // 2 + 1), nx, 2 * math.pi / lx)
        ky, oy, ey = waves(_modes(ny), ny, 2 * math.pi / ly)
        kz, oz, ez = waves(_modes(n), n, 2 * math.pi / (n * self.dz))
        self.kx, self.ky, self.kz = ox[None, None], oy[None, :, None], oz[:, None, None]
        self.k2 = kx[None, None] ** 2 + ky[None, :, None] ** 2 + kz[:, None, None] ** 2
        self.k2o = self.kx ** 2 + self.ky ** 2 + self.kz ** 2
        self.sigma = torch.exp(-16 * math.log(10.0) * (
            ((2 * ez) ** 100)[:, None, None] + ((2 * ey) ** 100)[None, :, None]
            + ((2 * ex) ** 100)[None, None]))
        self.gam = torch.sqrt(self.kx ** 2 + self.ky ** 2)[0]

    def extend(self, f):
        flat = f.reshape(f.shape[0], -1)
        m = self.m_r.to(flat.dtype)
        tail = m @ flat[-self.d:] + m.flip(0, 1) @ flat[:self.d]
        return torch.cat([flat, tail]).reshape((-1,) + f.shape[1:])

    def fz(self, m):
        return torch.fft.fft(self.extend(m), dim=0)

    def bz(self, s):
        return torch.fft.ifft(s, dim=0)[:self.nz]

    def fxy(self, a):
        return torch.fft.fft(torch.fft.rfft(a, dim=-1), dim=-2)

    def bxy(self, m):
        m = torch.fft.ifft(m, dim=-2)
        m[..., 0].imag.zero_()
        m[..., -1].imag.zero_()
        return torch.fft.irfft(m, n=self.nx, dim=-1)

    def nonlinear(self, w):
        vel = [self.bxy(self.bz(q)) for q in w[:3]]
        out = []
        for q in w:
            m = self.bz(q)
            out.append(-(vel[0] * self.bxy(1j * self.kx * m) + vel[1] * self.bxy(1j * self.ky * m)
                         + vel[2] * self.bxy(self.bz(1j * self.kz * q))))
        return out

    def project(self, vs, c):
        s = self.kx * vs[0] + self.ky * vs[1] + self.kz * vs[2]
        s = torch.where(self.k2o > 0, s / torch.where(self.k2o > 0, self.k2o, 1.0), 0.0 * s)
        r = self.bz(vs[2] - self.kz * s)
        b, t = r[0].clone(), r[-1].clone()
        del r
        pos, g = self.gam > 0, torch.where(self.gam > 0, self.gam, 1.0)
        e = torch.exp(-g * self.lz)
        den = g * (1 - e * e)
        zero = torch.zeros_like(b)
        ca, cb = torch.where(pos, (t - b * e) / den, zero), torch.where(pos, (t * e - b) / den, zero)
        cd = torch.where(pos, zero, 0.5 * (b + t))
        z = (torch.arange(self.nz, dtype=torch.float64, device=DEV) * self.dz)[:, None, None]
        pa, pb = ca * torch.exp(g * (z - self.lz)), cb * torch.exp(-g * z)
        sym = pa + pb
        hx, hy = 1j * self.kx * sym, 1j * self.ky * sym
        new = [vs[0] - self.kx * s - self.fz(hx), vs[1] - self.ky * s - self.fz(hy),
               vs[2] - self.kz * s - self.fz(self.gam * (pa - pb) + cd)]
        sm = self.bz(s)
        gw = torch.stack([torch.stack([self.kx[0] * sm[i] + hx[i], self.ky[0] * sm[i] + hy[i]])
                          for i in (0, self.nz - 1)]) / c
        return new, gw, self.bz(-1j * s) + sym + cd * z

    def solve(self, v, theta, dt, steps, order):
        vt = [self.fz(self.fxy(v[i])) for i in range(3)]
        if self.boussinesq:
            vt.append(self.fz(self.fxy(theta)))
        gw = torch.zeros((2, 2) + tuple(vt[0].shape[1:]), dtype=torch.complex128, device=DEV)
        phi, c = None, 1.0
        for _ in range(steps):
            w = vt
            for j in range(1, order + 1):
                c = dt / (order - j + 1)
                nl = self.nonlinear(w)
                st = []
                for f, q in enumerate(w):
                    k = self.kappa if f == 3 else self.nu
                    nf = self.sigma * self.fz(self.fxy(nl[f]))
                    st.append(self.bz(vt[f] + c * (nf - k * self.k2 * q)))
                    nl[f] = None
                st[0][:, 0, 0] += c * self.forcing_x * self.nx * self.ny
                if self.boussinesq:
                    st[2] += c * self.gamma * self.bz(w[3])
                    st[3] += c * self.gamma * self.bz(w[2])
                    st[3][0] = 0
                    st[3][-1] = 0
                for i in (0, 1):
                    st[i][0], st[i][-1] = c * gw[0, i], c * gw[1, i]
                vs = [self.fz(x) for x in st]
                new, gw, phi = self.project(vs[:3], c)
                w = new + vs[3:]
            vt = w
        phys = [self.bxy(self.bz(q)) for q in vt]
        pres = self.bxy(phi / c)
        return (vt, torch.stack(phys[:3]), phys[3] if self.boussinesq else None,
                pres - pres.mean())

    def statistics(self, vt, v, theta, zs):
        """The 13 flow diagnostics and the two 1D spectra of u at height index zs."""
        div = self.bxy(self.bz(1j * (self.kx * vt[0] + self.ky * vt[1] + self.kz * vt[2])))
        du = self.bxy(self.bz(1j * self.kz * vt[0]))
        d0, d1 = float(du[0].mean()), float(du[-1].mean())
        re = [math.sqrt(self.nu * abs(x)) * self.lz / 2 / self.nu for x in (d0, d1)]
        out = [0.5 * float(v.square().sum(0).mean()), float(div.square().mean())]
        out += [float((v[0, i] ** 2 + v[1, i] ** 2).mean()) for i in (0, -1)]
        out += [float((v[2, i] ** 2).mean()) for i in (0, -1)] + [d0, d1] + re
        if self.boussinesq:
            dt = self.bxy(self.bz(1j * self.kz * vt[3]))
            out += [1 - float(dt[i].mean()) / self.gamma for i in (0, -1)]
            out.append(float(theta.square().mean()))
        else:
            out += [math.nan, math.nan, 0.0]
        f = torch.fft.fft2(v[0, zs].to(torch.complex128)) / (self.nx * self.ny)
        e = f.abs() ** 2
        col = e.sum(0)
        h = self.nx // 2
        ex = col[:h + 1].clone()
        ex[1:h] += col[h + 1:].flip(0)
        return [np.array(out), ex.cpu().numpy(), e.sum(1).cpu().numpy()]


def _plain(c):
    return _Plain(c["nx"], c["ny"], c["nz"], c["C"], c["d"], **_physics(c))


def exact(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind == "serve":
        out = []
        for i, r in enumerate(_serve_requests(c)):
            v, th = _initial(r, seed * 100 + i)
            _, v, th, _ = _plain(r).solve(v, th, r["dt"], r["steps"], r["order"])
            out.append((v.cpu().numpy(), th.cpu().numpy() if th is not None else None))
        return out
    if kind in ("derivative", "extend"):
        q = _Plain(8, 8, c["nz"], c["C"], c["d"], 1.0, 1.0, 1.0, 1e-3)
        f = q.extend(_lines_input(c, seed).t().contiguous())
        if kind == "extend":
            return f.t().contiguous()
        f = torch.fft.fft(f.to(torch.complex128), dim=0)
        kz = q.kz[:, :, 0]
        if c["order"] == 1:
            f = f * (1j * kz)
        else:
            m = _modes(q.n).to(DEV, torch.float64)
            f = f * (-((m * (2 * math.pi / (q.n * q.dz))) ** 2))[:, None]
        return torch.fft.ifft(f, dim=0)[:c["nz"]].real.t().contiguous()
    q = _plain(c)
    if kind == "project":
        v = _project_input(c, seed)
        new, gw, _ = q.project([q.fz(q.fxy(v[i])) for i in range(3)], 1e-3)
        return (torch.stack([q.bxy(q.bz(x)) for x in new]), q.bxy(gw))
    if kind == "rhs":
        v, th = _rhs_input(c, seed)
        w = [q.fz(q.fxy(x)) for x in list(v) + ([th] if th is not None else [])]
        nl = q.nonlinear(w)
        if c["filtered"]:
            nl = [q.bxy(q.bz(q.sigma * q.fz(q.fxy(x)))) for x in nl]
        return (torch.stack(nl[:3]), nl[3] if th is not None else None)
    v, th = _initial(c, seed)
    vt, v, th, p = q.solve(v, th, c["dt"], c["steps"], c["order"])
    out = [v, th, p if c["pressure"] else None]
    if c["stats"]:
        out.extend(q.statistics(vt, v, th, c["nz"] // 2))
    return out
