"""Performance cases of the D3Q27 free-energy LB library: what a program that
uses it runs, through the public entry points (`lbfe.Simulation` and
`autograd.simulate`), over the range of grids, storage forms, boundaries and
directions that the library serves.

    listed()            the fixed cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) the program's state before the call, on the GPU
    run(state)          one pass and its outputs
    work(case)          bytes and flops that one pass cannot do without
    exact(case, seed)   the outputs of run in 64-bit plain torch, or None

Three kinds of pass:
    evolve    set an initial density (and velocity), step, read the result: the
              macroscopic fields in FP64, the raw checkpoint in the FP32 and
              FP16-deviation forms
    monitor   as evolve, with the mass, momentum, force and speed reductions
              read after every `every` steps, as a run that logs its invariants
    gradient  the differentiable simulation: density after `steps` steps and the
              gradients of a quadratic loss by the checkpointed reverse sweep
"""
import math

import torch
from torch.utils.checkpoint import checkpoint

from paper_2504_03819_amd import autograd, inputs, lbfe

A_EOS, B_EOS, KAPPA, NU = 9.0 / 392.0, 2.0 / 21.0, 0.02, 0.15
TC = 8.0 * A_EOS / (27.0 * B_EOS)
POP = {"fp64": 8, "fp32": 4, "fp16dev_f0fp32": 2}


def _case(name, kind, nx, ny, nz, precision, boundary, field, tr, steps, **kw):
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, precision=precision, boundary=boundary, field=field, tr=tr, steps=steps,
             wet_mode=kw.get("wet_mode", lbfe.WET_NEUTRAL), wet_value=kw.get("wet_value", 1.0),
             omega3=kw.get("omega3", 1.0), velocity=kw.get("velocity", 0.0), every=kw.get("every", 0))
    if name:
        c["name"] = name
    return c


def listed():
    walls = dict(omega3=0.5)
    return [
        # The smallest box of the paper's test problems, where every kernel of a
        # step is shorter than the time to start it: a stationary droplet.
        _case("droplet 32^3 fp64", "evolve", 32, 32, 32, "fp64", "periodic", "droplet", 0.9, 100),
        # A small phase separation that logs its invariants every ten steps:
        # short calls, each with its readback.
        _case("monitored 64^3 fp32", "monitor", 64, 64, 64, "fp32", "periodic", "spinodal", 0.8, 100, every=10),
        # An ordinary box between moving walls whose extents are odd and far from
        # any tile size.
        _case("moving walls 101x67x53 fp64", "evolve", 101, 67, 53, "fp64", "moving_walls", "droplet", 0.8, 30, **walls),
        # The moving droplet of the Galilean-invariance test, in both storage
        # widths: the ordinary production size.
        _case("droplet 128^3 fp64", "evolve", 128, 128, 128, "fp64", "periodic", "droplet", 0.85, 30, velocity=0.05),
        _case("droplet 128^3 fp32", "evolve", 128, 128, 128, "fp32", "periodic", "droplet", 0.85, 30, velocity=0.05),
        # The sessile droplet on a flat wall, the wetting studies' box.
        _case("wetting 192x192x96 fp32", "evolve", 192, 192, 96, "fp32", "walls", "droplet", 0.7, 30,
              wet_mode=lbfe.WET_PHI, wet_value=1.0, **walls),
        # A droplet on a pillared substrate: a solid voxel mask.
        _case("pillars 192x192x96 fp64", "evolve", 192, 192, 96, "fp64", "pillars", "droplet", 0.7, 20,
              wet_mode=lbfe.WET_DELTA, wet_value=0.9, **walls),
        # Spinodal decomposition in the narrow storage form: a large box of a
        # statistics run.
        _case("spinodal 256^3 fp16", "evolve", 256, 256, 256, "fp16dev_f0fp32", "periodic", "spinodal", 0.8, 20),
        # The largest box: two droplets colliding head-on, in both widths.
        _case("collision 512^3 fp64", "evolve", 512, 512, 512, "fp64", "periodic", "collision", 0.85, 10, velocity=0.04),
        _case("collision 512^3 fp32", "evolve", 512, 512, 512, "fp32", "periodic", "collision", 0.85, 10, velocity=0.04),
        # Gradients through a small wetting problem in FP64, and through the
        # wetting studies' box in FP32: the reverse sweep with its recomputation.
        _case("gradient 48x40x32 fp64", "gradient", 48, 40, 32, "fp64", "walls", "droplet", 0.7, 12,
              wet_mode=lbfe.WET_PHI, wet_value=1.28, **walls),
        _case("gradient 192x192x96 fp32", "gradient", 192, 192, 96, "fp32", "walls", "droplet", 0.7, 10,
              wet_mode=lbfe.WET_PHI, wet_value=1.0, **walls),
    ]


def draw(rng):
    """A case of the listed ranges: 2^12 to 2^24.5 nodes (gradients to 2^21.5),
    extents of any parity, every boundary and storage form in use."""
    kind = rng.choice(("evolve", "evolve", "evolve", "monitor", "gradient"))
    top = 21.5 if kind == "gradient" else 24.5
    nodes = 2.0 ** rng.uniform(12.0, top)
    side = nodes ** (1.0 / 3.0)
    ex, ey = math.exp(rng.uniform(-0.4, 0.4)), math.exp(rng.uniform(-0.4, 0.4))
    nx, ny = max(12, round(side * ex)), max(12, round(side * ey))
    nz = max(12, round(nodes / (nx * ny)))
    if rng.random() < 0.4:  # extents that come in round numbers
        nx, ny = max(16, nx // 16 * 16), max(16, ny // 16 * 16)
    boundary = rng.choice(("periodic", "periodic", "walls", "moving_walls", "pillars"))
    if boundary == "pillars":
        nz = max(24, nz)
    precision = rng.choice(("fp64", "fp32") if kind == "gradient" else ("fp64", "fp32", "fp16dev_f0fp32"))
    field = rng.choice(("droplet", "spinodal")) if boundary == "periodic" else "droplet"
    mode = rng.choice((lbfe.WET_NEUTRAL, lbfe.WET_PHI, lbfe.WET_DELTA)) if boundary != "periodic" else lbfe.WET_NEUTRAL
    value = {lbfe.WET_NEUTRAL: 1.0, lbfe.WET_PHI: round(rng.uniform(1.0, 1.4), 3),
             lbfe.WET_DELTA: round(rng.uniform(0.2, 0.9), 3)}[mode]
    steps = 8 if kind == "gradient" else rng.choice((10, 20, 30))
    return _case(None, kind, nx, ny, nz, precision, boundary, field, round(rng.uniform(0.75, 0.9), 3), steps,
                 wet_mode=mode, wet_value=value, omega3=1.0 if boundary == "periodic" else 0.5,
                 velocity=round(rng.uniform(0.0, 0.05), 4) if boundary == "periodic" and field == "droplet" else 0.0,
                 every=10 if kind == "monitor" else 0)


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _shape(c):
    return (c["nz"], c["ny"], c["nx"])


def _wall_u(c):
    return (0.1, 0.0, 0.1, 0.0) if c["boundary"] == "moving_walls" else (0.0, 0.0, 0.0, 0.0)


def _omega(c):
    return [1.0, 1.0, 1.0, c["omega3"]] + [1.0] * 7


def _coexistence(tr):
    """Densities of equal chemical potential and equal pressure of the van der
    Waals fluid at T = tr T_c (Newton's method on the pair)."""
    T = tr * TC
    mu = lambda r: T * (math.log(r / (1.0 - B_EOS * r)) + 1.0 / (1.0 - B_EOS * r)) - 2.0 * A_EOS * r
    p = lambda r: r * T / (1.0 - B_EOS * r) - A_EOS * r * r
    dmu = lambda r: T / (r * (1.0 - B_EOS * r) ** 2) - 2.0 * A_EOS  # dp/dr = r dmu/dr
    rl, rv = 0.75 / B_EOS, 0.03 / B_EOS
    for _ in range(200):
        f1, f2 = mu(rl) - mu(rv), p(rl) - p(rv)
        a, b = dmu(rl), -dmu(rv)
        det = a * rv * b - b * rl * a
        dl, dv = (f1 * rv * b - b * f2) / det, (a * f2 - f1 * rl * a) / det
        s = 1.0
        while not 0.0 < rv - s * dv < rl - s * dl < 1.0 / B_EOS:
            s *= 0.5
        rl, rv = rl - s * dl, rv - s * dv
    return rl, rv


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _solid(c):
    if c["boundary"] != "pillars":
        return None
    return torch.from_numpy(inputs.mask_pillars(_shape(c), plate=2, pitch=12, width=4, height=6))


def _fields(c, seed):
    """Initial density (nz, ny, nx) and velocity (3, nz, ny, nx) or None, and
    the coexistence pair: tanh droplets of width 5 (Eqs. (34)-(35)) with the
    seed's centre and a 1e-3 noise, or a noisy mean density."""
    dev = _device()
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    rl, rv = _coexistence(c["tr"])
    nz, ny, nx = _shape(c)
    f64 = dict(dtype=torch.float64, device=dev)
    noise = 2.0 * torch.rand(_shape(c), generator=g, **f64) - 1.0
    if c["field"] == "spinodal":
        return 0.5 * (rl + rv) * (1.0 + 0.01 * noise), None, rl, rv
    jit = (torch.rand(3, generator=g, **f64) - 0.5).tolist()
    z = torch.arange(nz, **f64)[:, None, None]
    y = torch.arange(ny, **f64)[None, :, None]
    x = torch.arange(nx, **f64)[None, None, :]

    def ball(cx, cy, cz, r):  # 0..1 indicator
        d = torch.sqrt((x - cx) ** 2 + (y - cy) ** 2 + (z - cz) ** 2)
        return 0.5 - 0.5 * torch.tanh(2.0 * (d - r) / 5.0)

    u = None
    if c["field"] == "collision":
        r, gap = nx / 8.0, nx * 160.0 / 512.0
        chi1 = ball(nx / 2 - gap / 2 + jit[0], ny / 2 + jit[1], nz / 2 + jit[2], r)
        chi2 = ball(nx / 2 + gap / 2 + jit[0], ny / 2 - jit[1], nz / 2 - jit[2], r)
        rho = rv + (rl - rv) * (chi1 + chi2)
        u = torch.zeros((3,) + _shape(c), **f64)
        u[0] = c["velocity"] * (chi1 - chi2)
    else:
        seat = {"walls": 0.5, "pillars": 8.0}.get(c["boundary"], nz / 2)
        r = max(3.0, min(nx, ny, nz if seat == nz / 2 else 2 * nz) / (4.0 if c["boundary"] != "walls" else 6.0))
        rho = rv + (rl - rv) * ball(nx / 2 + jit[0], ny / 2 + jit[1], seat + (jit[2] if seat == nz / 2 else 0.0), r)
        if c["velocity"]:
            u = torch.empty((3,) + _shape(c), **f64)
            for a, s in enumerate((1.0, 0.4, 0.0)):
                u[a] = c["velocity"] * s
    rho = rho * (1.0 + 1e-3 * noise)
    if c["boundary"] in ("walls", "moving_walls"):
        rho[0] = rv
        rho[-1] = rv
    solid = _solid(c)
    if solid is not None:
        rho[solid.to(dev) != 0] = rv
    return rho, u, rl, rv


def prepare(case, seed):
    rho, u, rl, rv = _fields(case, seed)
    walls = int(case["boundary"] in ("walls", "moving_walls"))
    if case["kind"] == "gradient":
        cfg = autograd.StepConfig(nx=case["nx"], ny=case["ny"], nz=case["nz"], steps=case["steps"],
                                  checkpoint_every=case["steps"], T=case["tr"] * TC, nu=NU, walls_z=walls,
                                  wet_mode=case["wet_mode"], precision=case["precision"], omega=_omega(case),
                                  wall_u=_wall_u(case), solid=_solid(case), u0=u)
        dt = torch.float64 if case["precision"] == "fp64" else torch.float32
        # leaves in the width of the run, as a training program holds them
        return dict(case=case, cfg=cfg, rho=rho.to(dt).clone().requires_grad_(True), target=_target(case, rho),
                    kappa=torch.tensor(KAPPA, dtype=torch.float64, requires_grad=True),
                    wet=torch.tensor(case["wet_value"], dtype=torch.float64, requires_grad=True))
    sim = lbfe.Simulation(device="cuda", nx=case["nx"], ny=case["ny"], nz=case["nz"], T=case["tr"] * TC, nu=NU,
                          kappa=KAPPA, walls_z=walls, wet_mode=case["wet_mode"], wet_value=case["wet_value"],
                          precision=case["precision"], omega=_omega(case), wall_u=_wall_u(case), solid=_solid(case))
    return dict(case=case, sim=sim, rho=rho, u=u)


def _target(c, rho):
    """The density that a gradient run is fitted to: the initial one smoothed
    along x (values inside the coexistence range)."""
    return 0.5 * rho + 0.25 * (torch.roll(rho, 1, 2) + torch.roll(rho, -1, 2))


# --------------------------------------------------------------------------
# the pass
# --------------------------------------------------------------------------
def run(state):
    c = state["case"]
    if c["kind"] == "gradient":
        rho_T = autograd.simulate(state["rho"], state["kappa"], state["wet"], state["cfg"])
        loss = ((rho_T - state["target"]) ** 2).sum()
        g = torch.autograd.grad(loss, (state["rho"], state["kappa"], state["wet"]))
        return {"rho": rho_T.detach(), "grad_rho": g[0], "grad_kappa": g[1], "grad_wet": g[2]}
    sim = state["sim"]
    sim.init_density(state["rho"], state["u"])
    logged = []
    if c["kind"] == "monitor":
        for _ in range(c["steps"] // c["every"]):
            sim.step(c["every"])
            logged.append(sim.reduce())
    else:
        sim.step(c["steps"])
    out = dict(sim.fields()) if c["precision"] == "fp64" else _unpack(c, sim.get_state())
    if logged:
        out["log"] = torch.tensor(logged, dtype=torch.float64)
    return out


def _unpack(c, raw):
    """The raw checkpoint in its storage types (views): FP32 populations, or
    26 half deviations per row and the FP32 rest populations."""
    n = c["nx"] * c["ny"] * c["nz"]
    if c["precision"] == "fp32":
        return {"f": raw.view(torch.float32)}
    h = (26 * 2 * n + 255) // 256 * 256
    return {"h": raw[:26 * 2 * n].view(torch.float16), "f0": raw[h:h + 4 * n].view(torch.float32)}


# --------------------------------------------------------------------------
# the least work
# --------------------------------------------------------------------------
def work(case):
    """Per step and fluid node 54 populations (27 read, 27 written; for a
    reverse step 81: adjoint and forward state read, adjoint written) and about
    1000 flops (a reverse step about 2500); the initial fields read and the
    outputs written once; per logged reduction one read of the populations."""
    c = case
    n = c["nx"] * c["ny"] * c["nz"]
    nf = c["nx"] * c["ny"] * (c["nz"] - 2) if c["boundary"] in ("walls", "moving_walls") else n
    if c["boundary"] == "pillars":
        nf = int((_solid(c) == 0).sum())
    per = 26 * 2 + 4 if c["precision"] == "fp16dev_f0fp32" else 27 * POP[c["precision"]]
    has_u = c["velocity"] > 0
    if c["kind"] == "gradient":
        s = 8 if c["precision"] == "fp64" else 4
        return {"bytes": nf * c["steps"] * (2 * per + 81 * s) + n * (2 * s + 16 + (24 if has_u else 0)),
                "flops": 3500.0 * nf * c["steps"]}
    out = 64 if c["precision"] == "fp64" else per
    logs = c["steps"] // c["every"] if c["every"] else 0
    return {"bytes": nf * (c["steps"] * 2 * per + logs * per) + n * (8 + out + (24 if has_u else 0)),
            "flops": 1000.0 * nf * c["steps"]}


# --------------------------------------------------------------------------
# the same in 64 bits, plain torch
# --------------------------------------------------------------------------
DIRS = [(x, y, z) for x in (-1, 0, 1) for y in (-1, 0, 1) for z in (-1, 0, 1)]
W1 = {-1: 1.0 / 6.0, 0: 2.0 / 3.0, 1: 1.0 / 6.0}
W27 = [W1[x] * W1[y] * W1[z] for x, y, z in DIRS]


def _at(g, c):  # g at x + c, periodic
    return torch.roll(g, (-c[2], -c[1], -c[0]), (-3, -2, -1))


def _axis(g, dim, a, b, c):  # a g(-1) + b g(0) + c g(+1) along one axis
    return a * torch.roll(g, 1, dim) + b * g + c * torch.roll(g, -1, dim)


def _smooth(g, dim):
    return _axis(g, dim, 1.0 / 6.0, 2.0 / 3.0, 1.0 / 6.0)


def _grad(g, a):  # isotropic d/dx_a, a = 0, 1, 2 for x, y, z
    dims = (-1, -2, -3)
    for b in range(3):
        g = _axis(g, dims[b], -0.5, 0.0, 0.5) if b == a else _smooth(g, dims[b])
    return g


class _Step:
    """One time step of the model (generalized equilibria, central moments,
    wetting boundary, halfway bounce-back) on populations (3, 3, 3, nz, ny, nx)."""

    def __init__(self, c, dev):
        self.c = c
        self.rl, self.rv = _coexistence(c["tr"])
        self.RT = c["tr"] * TC
        s = torch.ones(_shape(c), dtype=torch.float64, device=dev)
        if c["boundary"] in ("walls", "moving_walls"):
            s[0] = s[-1] = 0.0
        if c["boundary"] == "pillars":
            s[_solid(c).to(dev) != 0] = 0.0
        self.s, self.fluid = s, s > 0
        self.bounded = c["boundary"] != "periodic"
        self.den = _smooth(_smooth(_smooth(s, -1), -2), -3)
        self.w = _omega(c)

    def average(self, g):  # over fluid neighbours, 0 where there is none
        num = _smooth(_smooth(_smooth(torch.where(self.fluid, g, torch.zeros_like(g)), -1), -2), -3)
        ok = self.den > 1e-12
        return torch.where(ok, num / torch.where(ok, self.den, torch.ones_like(num)), torch.zeros_like(num))

    def wall_density(self, rho, wet):
        if not self.bounded:
            return rho
        lo, hi = 0.05 * self.rl + 0.95 * self.rv, 0.95 * self.rl + 0.05 * self.rv
        ave = self.average(rho)
        mod = ave
        if self.c["wet_mode"] == lbfe.WET_PHI:
            mod = torch.clamp(wet * ave, lo, hi)
        elif self.c["wet_mode"] == lbfe.WET_DELTA:
            mod = torch.clamp(ave - wet, lo, hi)
        return torch.where(self.fluid, rho, torch.where((ave >= lo) & (ave <= hi), mod, ave))

    def potential(self, rho, kappa):
        safe = torch.where(rho > 0, rho, torch.ones_like(rho))
        inv = 1.0 / (1.0 - B_EOS * safe)
        mu = self.RT * (torch.log(safe * inv) + inv) - 2.0 * A_EOS * safe
        mu = mu - 6.0 * kappa * (_smooth(_smooth(_smooth(rho, -1), -2), -3) - rho)
        return torch.where(self.fluid, mu, self.average(mu)) if self.bounded else mu

    def moments(self, f):
        rho = f.sum((0, 1, 2))
        j = []
        for a in range(3):
            m = f.sum([b for b in range(3) if b != a])
            j.append(m[2] - m[0])
        return rho, torch.stack(j)

    def fields(self, f, kappa, wet):
        rho, j = self.moments(f)
        rho = self.wall_density(rho, wet)
        mu = self.potential(rho, kappa)
        F = torch.stack([(1.0 / 3.0 - rho) * _grad(mu, a) * self.s for a in range(3)])
        safe = torch.where(self.fluid, rho, torch.ones_like(rho))
        u = (j + 0.5 * F) / safe * self.s
        return rho, mu, F, u, safe

    @staticmethod
    def _map(t, dim, A):  # t'_m = sum_c A[m][c] t_c along one of the first three axes
        p = t.unbind(dim)
        return torch.stack([A[m][0] * p[0] + A[m][1] * p[1] + A[m][2] * p[2] for m in range(3)], dim)

    @staticmethod
    def _shift(t, dim, u):  # raw to central moments by -u, and back by +u
        m0, m1, m2 = t.unbind(dim)
        return torch.stack([m0, m1 + u * m0, m2 + 2.0 * u * m1 + u * u * m0], dim)

    def to_central(self, f, u):
        for a in range(3):
            f = self._shift(self._map(f, a, ((1, 1, 1), (-1, 0, 1), (1, 0, 1))), a, -u[a])
        return f

    def to_populations(self, k, u):
        for a in range(3):
            k = self._map(self._shift(k, a, u[a]), a, ((0, -0.5, 0.5), (1, 0, -1), (0, 0.5, 0.5)))
        return k

    def equilibrium(self, rho, pm, u):
        z = torch.zeros_like(pm)
        k = [[[z for _ in range(3)] for _ in range(3)] for _ in range(3)]
        k[0][0][0] = rho
        k[2][0][0] = k[0][2][0] = k[0][0][2] = pm
        k[2][2][0] = k[2][0][2] = k[0][2][2] = pm / 3.0
        k[2][2][2] = pm / 9.0
        return self.to_populations(torch.stack([torch.stack([torch.stack(r) for r in p]) for p in k]), u)

    def __call__(self, f, kappa, wet):
        w = self.w
        rho, mu, F, u, safe = self.fields(f, kappa, wet)
        pm = (1.0 + mu) / 3.0
        Q = [-3.0 * _grad((pm - rho / 3.0) * u[a] * self.s, a) * self.s for a in range(3)]
        w1 = 1.0 / (safe * NU / pm + 0.5)
        k = self.to_central(f, u)
        o = {}
        for a, e in enumerate(((1, 0, 0), (0, 1, 0), (0, 0, 1))):
            o[e] = (1 - w[0]) * k[e] + (1 - w[0] / 2) * F[a]
        for e in ((1, 1, 0), (0, 1, 1), (1, 0, 1)):
            o[e] = (1 - w1) * k[e]
        xx, yy, zz = (2, 0, 0), (0, 2, 0), (0, 0, 2)
        d1 = (1 - w1) * (k[xx] - k[yy]) + (1 - w1 / 2) * (Q[0] - Q[1])
        d2 = (1 - w1) * (k[xx] - k[zz]) + (1 - w1 / 2) * (Q[0] - Q[2])
        tr = (1 - w[2]) * (k[xx] + k[yy] + k[zz]) + 3 * w[2] * pm + (1 - w[2] / 2) * (Q[0] + Q[1] + Q[2])
        o[xx], o[yy], o[zz] = (tr + d1 + d2) / 3, (tr - 2 * d1 + d2) / 3, (tr + d1 - 2 * d2) / 3
        for p, q, a in (((1, 2, 0), (1, 0, 2), 0), ((2, 1, 0), (0, 1, 2), 1), ((2, 0, 1), (0, 2, 1), 2)):
            sm = (1 - w[3]) * (k[p] + k[q]) + (1 - w[3] / 2) * (2.0 / 3.0) * F[a]
            df = (1 - w[4]) * (k[p] - k[q])
            o[p], o[q] = (sm + df) / 2, (sm - df) / 2
        o[1, 1, 1] = (1 - w[5]) * k[1, 1, 1]
        xy, xz, yz = (2, 2, 0), (2, 0, 2), (0, 2, 2)
        R = [(Q[0] + Q[1]) / 3, (Q[0] + Q[2]) / 3, (Q[1] + Q[2]) / 3]
        d1 = (1 - w[6]) * (k[xy] - 2 * k[xz] + k[yz]) + (1 - w[6] / 2) * (R[0] - 2 * R[1] + R[2])
        d2 = (1 - w[6]) * (k[xy] + k[xz] - 2 * k[yz]) + (1 - w[6] / 2) * (R[0] + R[1] - 2 * R[2])
        tr = (1 - w[7]) * (k[xy] + k[xz] + k[yz]) + w[7] * pm + (1 - w[7] / 2) * (R[0] + R[1] + R[2])
        o[xy], o[xz], o[yz] = (tr + d1 + d2) / 3, (tr - d1) / 3, (tr - d2) / 3
        for e in ((2, 1, 1), (1, 2, 1), (1, 1, 2)):
            o[e] = (1 - w[8]) * k[e]
        for a, e in enumerate(((1, 2, 2), (2, 1, 2), (2, 2, 1))):
            o[e] = (1 - w[9]) * k[e] + (1 - w[9] / 2) * F[a] / 9.0
        o[2, 2, 2] = (1 - w[10]) * k[2, 2, 2] + w[10] * pm / 9.0
        o[0, 0, 0] = k[0, 0, 0]
        ks = torch.stack([torch.stack([torch.stack([o[a, b, g] for g in range(3)]) for b in range(3)]) for a in range(3)])
        return self.stream(self.to_populations(ks, u), rho, pm)

    def stream(self, fs, rho, pm):
        moving = self.c["boundary"] == "moving_walls"
        if moving:
            uw = [torch.full_like(rho, v) for v in _wall_u(self.c)[:2]] + [torch.zeros_like(rho)]
            fe = self.equilibrium(rho, pm, uw)  # both walls move alike
        out = []
        for (x, y, z) in DIRS:
            v = _at(fs[x + 1, y + 1, z + 1], (-x, -y, -z))
            if self.bounded:
                back = fs[1 - x, 1 - y, 1 - z]
                if moving and z:
                    back = back - (fe[1 - x, 1 - y, 1 - z] - fe[x + 1, y + 1, z + 1])
                v = torch.where(_at(self.s, (-x, -y, -z)) > 0, v, back) * self.s
            out.append(v)
        return torch.stack(out).reshape(fs.shape)

    def initial(self, rho0, u0, kappa, wet):
        rho = self.wall_density(rho0, wet)
        pm = (1.0 + self.potential(rho, kappa)) / 3.0
        u = [torch.zeros_like(rho)] * 3 if u0 is None else [u0[a] * self.s for a in range(3)]
        f = self.equilibrium(torch.where(self.fluid, rho, torch.ones_like(rho)), pm, u)
        return f * self.s


def exact(case, seed):
    """Boxes up to 2^24.6 nodes (gradients up to 2^22); larger ones do not fit
    plain torch arrays."""
    c = case
    n = c["nx"] * c["ny"] * c["nz"]
    if n > (2 ** 22 if c["kind"] == "gradient" else 2 ** 24.6) or (not torch.cuda.is_available() and n > 2 ** 17):
        return None
    dev = _device()
    step = _Step(c, dev)
    rho, u, _, _ = _fields(c, seed)
    if c["kind"] == "gradient":
        dt = torch.float64 if c["precision"] == "fp64" else torch.float32
        target = _target(c, rho)
        r0 = rho.to(dt).double().requires_grad_(True)
        kap = torch.tensor(KAPPA, dtype=torch.float64, device=dev, requires_grad=True)
        wet = torch.tensor(c["wet_value"], dtype=torch.float64, device=dev, requires_grad=True)
        f = step.initial(r0, u, kap, wet)
        for _ in range(c["steps"]):
            f = checkpoint(step, f, kap, wet, use_reentrant=False)
        rho_T = step.wall_density(f.sum((0, 1, 2)), wet)
        # the loss sees the fluid densities: a solid node's density carries no gradient
        loss = (((rho_T - target) ** 2) * step.s).sum()
        g = torch.autograd.grad(loss, (r0, kap, wet), allow_unused=True)
        zero = torch.zeros((), dtype=torch.float64)
        return {"rho": rho_T.detach(), "grad_rho": g[0] * step.s, "grad_kappa": g[1].cpu(),
                "grad_wet": zero if g[2] is None else g[2].cpu()}
    log = []
    with torch.no_grad():
        kw = (KAPPA, c["wet_value"])
        f = step.initial(rho, u, *kw)
        for t in range(c["steps"]):
            f = step(f, *kw)
            if c["every"] and (t + 1) % c["every"] == 0:
                r, _, F, v, _ = step.fields(f, *kw)
                _, j = step.moments(f)
                log.append([float((r * step.s).sum())] + [float(a.sum()) for a in j] + [float(a.sum()) for a in F] +
                           [float(v.square().sum(0).sqrt().max())])
        if c["precision"] == "fp64":
            r, mu, F, v, _ = step.fields(f, *kw)
            out = {"rho": r, "u": v, "mu": mu, "F": F}
        else:
            p = f.reshape((27,) + _shape(c)).permute(1, 2, 0, 3)  # raw order [z][y][i][x]
            if c["precision"] == "fp32":
                out = {"f": p.reshape(-1)}
            else:
                wt = torch.tensor(W27, dtype=torch.float64, device=dev)[:, None]
                fl = step.s[:, :, None, :]
                h = ((p - wt) / wt) * fl
                out = {"h": torch.cat((h[:, :, :13], h[:, :, 14:]), 2).reshape(-1), "f0": p[:, :, 13].reshape(-1)}
    if log:
        out["log"] = torch.tensor(log, dtype=torch.float64)
    return out
