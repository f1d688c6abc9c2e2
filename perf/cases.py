"""Workloads that time the solver as its users run it.

A pass of a "run" case is what a study does again and again: load the start
state, advance a number of steps, read the probe histories, the diagnostics
and the fluid state. A "sweep" case does it for a batch of uneven instances,
an "adjoint" case takes the impulse and its gradient from the loaded state.
The solver's state is single precision on the GPU (fluid() and the readers
hand its values out in double precision arrays), so a pass returns what it
read in single precision.

The start states are seeded: the set-up lattice displaced around a disk that
is half way through its velocity ramp, a smooth random velocity and density
field (tens of m/s, about 1.5 % or 30 MPa) over the whole channel, so that
walls, probes and every pair see the pressures of a developed run.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2609_05494_amd as wc
import workloads

T0 = 2.5e-6  # time of the start state: half of the 5 us velocity ramp


# -- cases --------------------------------------------------------------------
def _case(name, kind, L, W, dx, R, v0, steps, **opt):
    """A planar single-instance case; `opt`: options of the workload (see _config) and the adjoint's ckpt."""
    c = dict(kind=kind, L=L, W=W, dx=dx, R=R, v0=v0, steps=steps)
    c.update(opt)
    if name:
        c["name"] = name
    return c


def listed():
    mm = 1e-3
    return [
        # one step at a time of a channel of a few hundred particles: an interactive loop, or a debugger's
        _case("tiny_1step", "run", 24 * mm, 16 * mm, 1 * mm, 3 * mm, 300.0, 1),
        # the smallest configured channel: a quick look at a parameter, launch latency and little else
        _case("channel_80", "run", 80 * mm, 40 * mm, 1 * mm, 4 * mm, 600.0, 60),
        # the gradient study's channel, stepped forward only (its finite-difference runs)
        _case("channel_120", "run", 120 * mm, 60 * mm, 0.5 * mm, 6 * mm, 900.0, 60),
        # the headline channel, 179,552 particles
        _case("channel_300", "run", 300 * mm, 150 * mm, 0.5 * mm, 6 * mm, 900.0, 60),
        # the largest configured channel, 719,552 particles
        _case("channel_600", "run", 600 * mm, 300 * mm, 0.5 * mm, 6 * mm, 900.0, 40),
        # the free disk with the energy audit, on a channel that is no multiple of anything; a step count that
        # is no multiple of the diagnostic interval
        _case("two_way_audit", "run", 203 * mm, 97 * mm, 0.7 * mm, 5 * mm, 750.0, 47, two_way=True, audit=True),
        # the paper's production channel with its own scheme (summation density, leapfrog, internal energy)
        _case("paper_scheme", "run", 750 * mm, 150 * mm, 1.5 * mm, 6.25 * mm, 900.0, 60, paper=True),
        # the same channel's cubic kernel and single-line walls, Mie-Grueneisen EOS, quadratic artificial viscosity
        _case("cubic_mg", "run", 401 * mm, 99 * mm, 0.9 * mm, 6.25 * mm, 900.0, 50, cubic=True, mg=True, beta=1.0),
        # the tank in the r-z form
        _case("axisymmetric", "run", 300 * mm, 150 * mm, 0.5 * mm, 6 * mm, 900.0, 50, axisym=True),
        # the coefficient sweep: sixteen instances of different length, alpha, delta and speed in one batch
        dict(name="sweep_16", kind="sweep", n_inst=16, W=100 * mm, dx=1 * mm, R=4 * mm, steps=60),
        # impulse and gradient with the whole run taped
        _case("adjoint_taped", "adjoint", 120 * mm, 60 * mm, 0.5 * mm, 6 * mm, 900.0, 40, ckpt=40),
        # the same through checkpoints, on a smaller odd channel
        _case("adjoint_ckpt", "adjoint", 77 * mm, 31 * mm, 0.6 * mm, 4 * mm, 600.0, 50, ckpt=10),
    ]


def draw(rng):
    """One more case over the listed ranges: 1,500 to 350,000 fluid particles, any aspect, spacing, option and step count."""
    kind = rng.choices(("run", "sweep", "adjoint"), (7, 2, 1))[0]
    dx = round(math.exp(rng.uniform(math.log(0.4e-3), math.log(1.6e-3))), 6)
    v0 = round(rng.uniform(300.0, 900.0), 1)
    if kind == "sweep":
        return dict(kind=kind, n_inst=rng.randint(2, 14), W=round(rng.uniform(0.04, 0.1), 4), dx=round(max(dx, 1e-3), 6),
                    R=4e-3, steps=rng.randint(20, 60))
    nf = math.exp(rng.uniform(math.log(1500.0), math.log(350000.0 if kind == "run" else 40000.0)))
    aspect = rng.uniform(1.3, 5.0)
    W = round(max(dx * math.sqrt(nf / aspect), 16 * dx), 5)
    L = round(dx * dx * nf / W, 5)
    R = round(min(0.2 * W, rng.uniform(4.0, 12.0) * dx), 6)
    if kind == "adjoint":
        return _case(None, kind, L, W, dx, R, v0, rng.randint(10, 40), ckpt=rng.choice((7, 40)))
    opt = rng.choice(({}, {}, {}, {"two_way": True}, {"audit": True}, {"paper": True}, {"cubic": True}, {"mg": True},
                      {"beta": 1.0}, {"axisym": True}))
    return _case(None, kind, L, W, dx, R, v0, rng.randint(10, 60), **opt)


# -- inputs ---------------------------------------------------------------------
def _config(c):
    cfg = workloads.base(c["L"], c["W"], c["dx"], c["R"], c["v0"], probes_x=(0.2 * c["L"], 0.6 * c["L"]))
    if c.get("cubic") or c.get("paper"):
        cfg = dict(cfg, kernel_type=1, ghost_layers=1, alpha=0.03)
    if c.get("mg"):
        cfg = workloads.mie_grueneisen(cfg)
    if c.get("beta"):
        cfg = dict(cfg, beta=c["beta"])
    if c.get("paper"):
        cfg = workloads.paper_scheme(cfg)
    if c.get("audit"):
        cfg = dict(cfg, audit=1)
    if c.get("two_way"):
        cfg = workloads.two_way(cfg)
    if c.get("axisym"):
        cfg = workloads.axisymmetric(cfg)
    return cfg


def _lattice(cfg):
    """The set-up lattice in particle-id order, the disk's interior removed."""
    dx = cfg["dx"]
    nx, ny = round(cfg["L"] / dx), round(cfg["W"] / dx)
    x = np.tile((np.arange(nx) + 0.5) * dx, ny)
    y = np.repeat((np.arange(ny) + 0.5) * dx, nx)
    keep = (x - cfg["disk_x0"]) ** 2 + (y - cfg["disk_y0"]) ** 2 >= cfg["disk_R"] ** 2
    return x[keep], y[keep]


def _fluid(cfg, seed):
    """The seeded start state at T0 (see above): x, y, vx, vy, rho."""
    r = np.random.default_rng(seed)
    x, y = _lattice(cfg)
    dx, R, n = cfg["dx"], cfg["disk_R"], x.size
    vd = cfg["kin_v0"] * T0 / cfg["kin_t_ramp"]
    shift = 0.5 * cfg["kin_v0"] * T0 * T0 / cfg["kin_t_ramp"]

    def field(rms):
        f = np.zeros(n)
        for _ in range(6):
            kx, ky = 2 * np.pi * r.uniform(0.5, 6.0, 2) / np.array([cfg["L"], cfg["W"]])
            f += np.cos(kx * x + ky * y * r.choice((-1, 1)) + r.uniform(0, 2 * np.pi))
        return f * (rms / math.sqrt(3.0))

    d = np.hypot(x - cfg["disk_x0"], y - cfg["disk_y0"])
    f = np.exp(-(d - R) / (2 * R))
    # compression of the map x -> x + shift f, kept below 8 %
    comp = np.clip(shift * f * (x - cfg["disk_x0"]) / (2 * R * np.maximum(d, dx)), -0.02, 0.08)
    vx, vy = vd * f + field(25.0), field(25.0)
    rho = cfg["rho0"] * (1.0 + comp + field(0.015))
    x = np.clip(x + shift * f + r.uniform(-0.05, 0.05, n) * dx, 0.1 * dx, cfg["L"] - 0.1 * dx)
    y = np.clip(y + r.uniform(-0.05, 0.05, n) * dx, 0.1 * dx, cfg["W"] - 0.1 * dx)
    return x, y, vx, vy, rho


def _sweep(c, seed):
    """Coefficient-sweep instances of the configured sweep's ranges (the lengths drawn once, the coefficients
    by the seed), with two probes ahead of the disk (the runs are short: the walls hear nothing yet)."""
    lengths = np.random.default_rng(workloads.C4_SEED).integers(200, 401, c["n_inst"])
    r = np.random.default_rng(seed)
    out = []
    for L in lengths:
        u = r.random(3)
        cfg = workloads.base(float(L) * 1e-3, c["W"], c["dx"], c["R"], 600.0 + 300.0 * u[2],
                             alpha=0.01 + 0.49 * u[0], delta=0.2 * u[1])
        out.append(dict(cfg, probes=[(0.012, 0.5 * c["W"]), (0.010, 0.5 * c["W"] + 0.004)]))
    return out


def prepare(case, seed):
    if case["kind"] == "sweep":
        s = wc.Solver(_sweep(case, seed), "cuda:0")
        return dict(case=case, s=s, blob=s.save_state())
    cfg = _config(case)
    s = wc.Solver(cfg, "cuda:0")
    if case["kind"] == "adjoint":
        # the fixed steps that the gradient is taken at: the CFL gate at the disk's speed
        s.set_dt_table(np.full(case["steps"], cfg["cfl"] * cfg["h_over_dx"] * cfg["dx"] / (cfg["c0"] + case["v0"])))
    s.set_fluid(T0, *_fluid(cfg, seed))
    return dict(case=case, s=s, blob=s.save_state())


# -- a pass -----------------------------------------------------------------------
def _f32(a):
    return np.asarray(a, dtype=np.float32)


def _diagnostics(d):
    """Diagnostic records as one table [record, quantity]."""
    return _f32(np.stack([d[k] for k in sorted(d)], axis=1))


def run(state):
    c, s = state["case"], state["s"]
    s.load_state(state["blob"])
    out = {}
    if c["kind"] == "adjoint":
        out["J"] = _f32(s.adj_forward(c["steps"], c["ckpt"]))
        out["grad"] = _f32(s.adj_backward(1.0))
    else:
        s.step(c["steps"])
    if c["kind"] == "sweep":
        # a sweep's product is its histories; a state is looked at one instance at a time
        probes, diags = [], []
        for i in range(s.n_inst):
            t, dt, p = s.read_probes(i)
            probes.append((t, dt, p))
            diags.append(_diagnostics(s.read_diagnostics(i)))
        out["t"], out["dt"], out["p"] = (_f32(np.stack([q[k] for q in probes])) for k in range(3))
        out["diagnostics"] = np.stack(diags)
        t, fluid = s.fluid(s.n_inst - 1)
    else:
        if c["kind"] == "run":
            t, dt, p = s.read_probes()
            out["t"], out["dt"], out["p"] = _f32(t), _f32(dt), p
            out["diagnostics"] = _diagnostics(s.read_diagnostics())
        if c.get("paper"):
            out["e"] = _f32(s.internal_energy())
        t, fluid = s.fluid()
    for k, v in zip(("x", "y", "vx", "vy", "rho"), fluid):
        out[k] = _f32(v)
    return out


# -- what a pass cannot do without ------------------------------------------------
def _fluid_count(c):
    if c["kind"] == "sweep":
        return c["n_inst"] * 0.3 * c["W"] / (c["dx"] * c["dx"])  # mean length 300 mm
    return _lattice(_config(c))[0].size


def work(case):
    """Bytes: the state in and out once per evaluation (32 B of position, velocity, density and mass in, 20 B
    out), and the loaded and the returned state. Flops: per evaluation 20 neighbours of 53 and 59 candidates of 5 per particle;
    the reverse sweep about twice its forward."""
    nf, k = _fluid_count(case), case["steps"]
    evals = k * (1 if case.get("paper") else 2) * (3 if case["kind"] == "adjoint" else 1)
    return {"bytes": nf * (52.0 * evals + 40.0), "flops": nf * evals * (20 * 53.0 + 59 * 5.0)}


# -- the same in 64 bits ------------------------------------------------------------
def exact(case, seed):
    """The fluid state after the pass by plain torch in float64: the planar predictor-corrector with a
    prescribed disk. The other forms (scheme 1, r-z, two-way disk, batch, gradient) are not restated here.
    Histories and records are a few reduced values each, left to the comparison of the two sides."""
    if case["kind"] != "run" or case.get("paper") or case.get("axisym") or case.get("two_way"):
        return None
    cfg = _config(case)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    S = _Reference(cfg, dev)
    u = [torch.tensor(v, dtype=torch.float64, device=dev) for v in _fluid(cfg, seed)]
    u = S.advance(T0, u, case["steps"])
    out = {k: None for k in ("t", "dt", "p", "diagnostics")}
    out.update({k: v.cpu() for k, v in zip(("x", "y", "vx", "vy", "rho"), u)})
    return out


class _Reference:
    """The step written down plainly in float64 (positions, velocities and density as five vectors)."""

    def __init__(self, cfg, dev):
        self.c, self.dev = cfg, dev
        dx = cfg["dx"]
        self.h = cfg["h_over_dx"] * dx
        nx, ny, g = round(cfg["L"] / dx), round(cfg["W"] / dx), cfg["ghost_layers"]
        i = torch.arange(-g, nx + g, device=dev, dtype=torch.float64)
        j = torch.arange(-g, ny + g, device=dev, dtype=torch.float64)
        jj, ii = torch.meshgrid(j, i, indexing="ij")
        wall = ~((ii >= 0) & (ii < nx) & (jj >= 0) & (jj < ny))
        self.wx, self.wy = (ii[wall] + 0.5) * dx, (jj[wall] + 0.5) * dx
        th = 2 * math.pi * torch.arange(cfg["n_disk_ghosts"], device=dev, dtype=torch.float64) / cfg["n_disk_ghosts"]
        self.ring = torch.cos(th), torch.sin(th)
        self.m = cfg["rho0"] * dx * dx
        self.m_disk = cfg["rho0"] * dx * 2 * math.pi * cfg["disk_R"] / cfg["n_disk_ghosts"]

    def disk(self, t):
        c = self.c
        v0, tr, x0 = c["kin_v0"], c["kin_t_ramp"], c["disk_x0"]
        if t < tr:
            return x0 + 0.5 * v0 * t * t / tr, v0 * t / tr, v0 / tr
        s, a = t - tr, c["kin_coef"]
        return x0 + 0.5 * v0 * tr + v0 * s - 0.5 * a * s * s, v0 - a * s, -a

    def eos(self, rho):
        c = self.c
        mu = rho / c["rho0"] - 1.0
        if c["eos_type"] == 1:
            mu = mu.clamp(max=c["mg_mu_max"])
            b, k1, K = c["mg_s1"] - 1.0, 1.0 - 0.5 * c["mg_gamma0"], c["rho0"] * c["c0"] ** 2
            up = mu >= 0
            den = torch.where(up, 1.0 - b * mu, torch.ones_like(mu))
            p = torch.where(up, K * mu * (1 + k1 * mu) / den ** 2, K * mu)
            cs = torch.where(up, c["c0"] * torch.sqrt(((1 + (2 * k1 + b) * mu) / den ** 3).clamp(min=0)),
                             torch.full_like(mu, c["c0"]))
        else:
            p = c["rho0"] * c["c0"] ** 2 / c["gamma"] * ((1 + mu) ** c["gamma"] - 1)
            cs = c["c0"] * (1 + mu) ** (0.5 * (c["gamma"] - 1))
        return p.clamp(min=c["p_cav"]), cs

    def kernel(self, r2):
        """W and (1/r) dW/dr."""
        h, q = self.h, torch.sqrt(r2) / self.h
        if self.c.get("kernel_type", 0) == 0:
            s = 1 - 0.5 * q
            return 7 / (4 * math.pi * h * h) * s ** 4 * (2 * q + 1), -35 / (4 * math.pi * h ** 4) * s ** 3
        a, s, near = 10 / (7 * math.pi * h * h), 2 - q, q <= 1
        W = torch.where(near, a * (1 - 1.5 * q * q + 0.75 * q ** 3), 0.25 * a * s ** 3)
        return W, a / (h * h) * torch.where(near, 2.25 * q - 3, -0.75 * s * s / torch.where(near, torch.ones_like(q), q))

    def pairs(self, ax, ay, bx, by):
        """Index pairs (a, b) closer than 2h."""
        e = 2.0 * self.h * (1 + 1e-9)
        g = self.c["ghost_layers"] * self.c["dx"] + e
        ncx = int((self.c["L"] + 2 * g) / e) + 2
        key = lambda x, y: torch.floor((y + g) / e).long() * ncx + torch.floor((x + g) / e).long()  # noqa: E731
        kb, order = torch.sort(key(bx, by))
        ka = key(ax, ay)
        ia, ib = [], []
        for row in (-1, 0, 1):
            k = ka + row * ncx
            lo, hi = torch.searchsorted(kb, k - 1), torch.searchsorted(kb, k + 1, right=True)
            n = hi - lo
            a = torch.repeat_interleave(torch.arange(len(ax), device=self.dev), n)
            first = torch.cumsum(n, 0) - n
            b = order[torch.arange(len(a), device=self.dev) - first[a] + lo[a]]
            near = (ax[a] - bx[b]) ** 2 + (ay[a] - by[b]) ** 2 < 4 * self.h ** 2
            ia.append(a[near])
            ib.append(b[near])
        return torch.cat(ia), torch.cat(ib)

    def rates(self, t, u):
        """Density rate, acceleration, XSPH correction and the largest speed of fluid and ghosts at state u."""
        c, h = self.c, self.h
        x, y, vx, vy, rho = u
        p, cs = self.eos(rho)
        xd, vd, ad = self.disk(t)
        gx = torch.cat([self.wx, xd + c["disk_R"] * self.ring[0]])
        gy = torch.cat([self.wy, c["disk_y0"] + c["disk_R"] * self.ring[1]])
        nw = len(self.wx)
        moving = torch.arange(len(gx), device=self.dev) >= nw
        # ghosts: Shepard averages of the fluid
        g, f = self.pairs(gx, gy, x, y)
        dx_, dy_ = gx[g] - x[f], gy[g] - y[f]
        W, _ = self.kernel(dx_ ** 2 + dy_ ** 2)
        add = lambda v: torch.zeros(len(gx), dtype=torch.float64, device=self.dev).index_add_(0, g, v)  # noqa: E731
        sw = add(W)
        has = sw > 0
        inv = torch.where(has, 1 / sw.clamp(min=1e-300), torch.zeros_like(sw))
        gp = (add(p[f] * W) - torch.where(moving, ad, 0.0) * add(rho[f] * dx_ * W)
              + c["gravity_y"] * add(rho[f] * dy_ * W)) * inv
        gp = gp.clamp(min=c["p_cav"])
        gvx = torch.where(has, 2 * torch.where(moving, vd, 0.0) - add(vx[f] * W) * inv, torch.where(moving, vd, 0.0))
        gvy = torch.where(has, -add(vy[f] * W) * inv, torch.zeros_like(sw))
        grho = c["rho0"] * (1 + gp / (c["rho0"] * c["c0"] ** 2))
        gc = self.eos(grho)[1]
        gm = torch.where(moving, self.m_disk, self.m)
        # pair sums over fluid and ghosts
        nf = len(x)
        X, Y, VX, VY = (torch.cat(q) for q in ((x, gx), (y, gy), (vx, gvx), (vy, gvy)))
        R, C, P = torch.cat([rho, grho]), torch.cat([cs, gc]), torch.cat([p / rho ** 2, gp / grho ** 2])
        M = torch.cat([torch.full_like(x, self.m), gm])
        i, j = self.pairs(x, y, X, Y)
        other = i != j
        i, j = i[other], j[other]
        rx, ry, ux, uy = X[i] - X[j], Y[i] - Y[j], VX[i] - VX[j], VY[i] - VY[j]
        r2 = rx ** 2 + ry ** 2
        W, F = self.kernel(r2)
        vr, fl = ux * rx + uy * ry, j < nf
        den, rs = r2 + c["eta2"] * h * h, R[i] + R[j]
        mu = h * vr.clamp(max=0) / den
        av = (-c["alpha"] * 0.5 * (C[i] + C[j]) * mu + c.get("beta", 0.0) * mu * mu) / (0.5 * rs)
        lam = 4 * c["mu_dyn"] / c["rho0"] * M[j] * F * r2 / (den * rs)
        s = M[j] * F * (P[i] + P[j] + av)
        delta = torch.where(fl, 2 * c["delta"] * h * c["c0"] * M[j] / R[j] * (R[i] - R[j]) * F, 0.0)
        xs = torch.where(fl, c["eps_xsph"] * 2 * M[j] / rs * W, 0.0)
        tot = lambda v: torch.zeros(nf, dtype=torch.float64, device=self.dev).index_add_(0, i, v)  # noqa: E731
        vmax = max(float(torch.hypot(vx, vy).max()), float(torch.hypot(gvx, gvy).max()))
        return (tot(M[j] * F * vr + delta), tot(lam * ux - s * rx), tot(lam * uy - s * ry) + c["gravity_y"],
                tot(-xs * ux), tot(-xs * uy), vmax)

    def enforce(self, x, y, vx, vy, t):
        c, e = self.c, self.c["eps_wall"]
        for v, w, hi in ((x, vx, c["L"]), (y, vy, c["W"])):
            out = (v < e) | (v > hi - e)
            w[out] = -w[out]
            v.clamp_(e, hi - e)
        xd, vd, _ = self.disk(t)
        rx, ry = x - xd, y - c["disk_y0"]
        d = torch.hypot(rx, ry)
        k = d < c["disk_R"]
        nx, ny = rx[k] / d[k], ry[k] / d[k]
        x[k], y[k] = xd + (c["disk_R"] + e) * nx, c["disk_y0"] + (c["disk_R"] + e) * ny
        w = ((vx[k] - vd) * nx + vy[k] * ny).clamp(max=0)
        vx[k] -= 2 * w * nx
        vy[k] -= 2 * w * ny

    def advance(self, t, u, steps):
        c = self.c
        lo, hi = c["rho_lo"] * c["rho0"], c["rho_hi"] * c["rho0"]
        for _ in range(steps):
            x, y, vx, vy, rho = u
            D, ax, ay, wx, wy, vmax = self.rates(t, u)
            dt = c["cfl"] * self.h / (c["c0"] + vmax)
            s = 0.5 * dt
            p = [x + s * (vx + wx), y + s * (vy + wy), vx + s * ax, vy + s * ay, (rho + s * D).clamp(lo, hi)]
            self.enforce(*p[:4], t + s)
            D, ax, ay, wx, wy, _ = self.rates(t + s, p)
            u = [x + dt * (p[2] + wx), y + dt * (p[3] + wy), vx + dt * ax, vy + dt * ay, (rho + dt * D).clamp(lo, hi)]
            t += dt
            self.enforce(*u[:4], t)
        return u
