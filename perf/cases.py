"""Performance cases of the dust hot path: what a run that uses this library
has it do, through the calls of ``paper_1908_10793_amd.dust``.

A gas code calls the library once per gas step (the predictor's drag source,
then one coupled step), so most cases are single calls of one step; a run of
test particles in a prescribed gas takes several steps per call.  The sizes
are those of the benchmark and of the tests, with ragged ones between.

  listed()      the named cases
  draw(rng)     one more case of the same ranges
  prepare()     inputs on the GPU, the context
  run()         one pass through the library
  work()        the bytes and operations that one pass cannot do without
  exact()       the pass in 64 bits, in plain torch
"""
import math

import numpy as np
import torch

from paper_1908_10793_amd import dust

TWO_PI = 2.0 * math.pi
SHEAR = dict(Omega=1.0, q=1.5)
TAUS = (0.01, 0.1, 1.0, 10.0)      # species of the periodic boxes


def listed():
    return [
        # the smallest run: a 2-D box in FP64, where launches and latency count
        dict(name="square_f64", call="step", grid="square", n0=64, n1=64, n2=1, ppc=16, prec="f64", shape="cic",
             drag="species", nsteps=1, rebin=1, feedback=True, det=False),
        # a small shearing box, one step per gas step
        dict(name="shear_32", call="step", grid="shear", n0=32, n1=32, n2=32, ppc=8, prec="f32", shape="tsc",
             drag="species", nsteps=1, rebin=1, feedback=True, det=False),
        # the benchmark's shearing box, one step per gas step
        dict(name="shear_128", call="step", grid="shear", n0=128, n1=128, n2=128, ppc=8, prec="f32", shape="tsc",
             drag="species", nsteps=1, rebin=1, feedback=True, det=False),
        # a batch of periodic boxes with four species: several steps per call (the largest)
        dict(name="batch_boxes", call="step", grid="boxes", sizes="32,48,64,80,96", ppc=66, prec="f32", shape="tsc",
             drag="species", nsteps=8, rebin=8, feedback=True, det=False),
        # the benchmark's cylindrical disk: log radii, Stokes numbers, a mass per particle
        dict(name="cyl_disk", call="step", grid="cyl", n0=256, n1=512, n2=64, ppc=4, prec="f32", shape="tsc",
             drag="stokes", nsteps=1, rebin=1, feedback=False, det=False),
        # a spherical disk of odd sizes with stiff stopping times
        dict(name="sph_disk", call="step", grid="sph", n0=131, n1=67, n2=259, ppc=4, prec="f32", shape="tsc",
             drag="tau", nsteps=1, rebin=1, feedback=False, det=False),
        # Epstein drag, which the unfused step alone takes
        dict(name="epstein_disk", call="unfused", grid="cyl", n0=128, n1=255, n2=33, ppc=4, prec="f32", shape="tsc",
             drag="epstein", nsteps=1, rebin=1, feedback=True, det=False),
        # a validation run: orbital advection in FP64
        dict(name="fargo_f64", call="step", grid="fargo", n0=64, n1=64, n2=64, ppc=8, prec="f64", shape="tsc",
             drag="species", nsteps=1, rebin=1, feedback=True, det=False),
        # what one gas step asks for in a shearing box: the predictor's source, then the step
        dict(name="cycle_shear", call="cycle", grid="shear", n0=100, n1=96, n2=72, ppc=8, prec="f32", shape="tsc",
             drag="species", nsteps=1, rebin=1, feedback=True, det=False),
        # the predictor's source in a disk, particles in the order that a step leaves
        dict(name="source_disk", call="source", grid="cyl", n0=192, n1=384, n2=48, ppc=4, prec="f32", shape="tsc",
             drag="stokes", nsteps=1, rebin=1, feedback=False, det=False),
        # the dust density of a snapshot (particles by cell, as written), four species
        dict(name="density_box", call="density", grid="boxes", sizes="96", ppc=34, prec="f32", shape="tsc",
             drag="species", nsteps=1, rebin=1, feedback=False, det=False),
        # a program that composes the step from the stage calls
        dict(name="stages_box", call="stages", grid="boxes", sizes="63", ppc=34, prec="f32", shape="tsc",
             drag="species", nsteps=1, rebin=1, feedback=True, det=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["square", "shear", "shear", "boxes", "cyl", "sph", "fargo", "epstein", "cycle", "source",
                       "density", "stages"])
    c = dict(call="step", prec="f32", shape=rng.choice(["tsc", "tsc", "tsc", "cic"]), drag="species", nsteps=1,
             rebin=1, feedback=True, det=False)
    if kind == "square":
        n = _log_int(rng, 24, 400)
        c.update(grid="square", n0=n, n1=max(8, n + rng.randint(-9, 9)), n2=1, ppc=rng.choice([4, 9, 16]),
                 prec=rng.choice(["f64", "f32"]))
    elif kind in ("shear", "cycle", "fargo"):
        n = _log_int(rng, 20, 72 if kind == "fargo" else 128)
        c.update(grid="fargo" if kind == "fargo" else "shear", n0=n, n1=max(16, n + rng.randint(-7, 7)),
                 n2=max(8, n // rng.choice([1, 2]) + rng.randint(-3, 3)), ppc=rng.choice([4, 8, 11]))
        c.update(call="cycle" if kind == "cycle" else "step",
                 prec="f64" if kind == "fargo" and rng.random() < 0.7 else "f32")
    elif kind in ("boxes", "density", "stages"):
        n = _log_int(rng, 24, 80)
        sizes = [n] if kind != "boxes" else [n, max(16, n - rng.randint(3, 20)), max(16, n // 2 + rng.randint(0, 5))]
        c.update(grid="boxes", sizes=",".join(str(s) for s in sizes), ppc=rng.choice([18, 34, 66]))
        if kind == "boxes":
            k = rng.choice([1, 2, 4, 8])
            c.update(nsteps=k, rebin=rng.choice([k, max(1, k // 2)]))
        else:
            c.update(call=kind, feedback=kind == "stages", det=kind == "stages" and rng.random() < 0.25)
    else:
        grid = rng.choice(["cyl", "sph"]) if kind in ("epstein", "source") else kind
        n = _log_int(rng, 24, 128)
        ncell2 = dict(cyl=(2 * n + rng.randint(-5, 5), max(8, n // 4 + rng.randint(-2, 2))),
                      sph=(max(12, n // 2 + rng.randint(-3, 3)), 2 * n + rng.randint(-5, 5)))[grid]
        c.update(grid=grid, n0=n, n1=ncell2[0], n2=ncell2[1], ppc=rng.choice([2, 4, 7]), feedback=False,
                 drag="stokes" if grid == "cyl" else "tau")
        if kind == "epstein":
            c.update(call="unfused", drag="epstein", feedback=True, det=rng.random() < 0.25)
        if kind == "source":
            c.update(call="source")
    return c


# ------------------------------------------------------------------ the grid and the gas

def _disk(R, z, p=-1.0, q=-0.5, h0=0.1):
    """Density and angular velocity of the disk gas in equilibrium (GM = 1)."""
    r = torch.sqrt(R * R + z * z)
    omk = R ** -1.5
    h = h0 * R ** ((q + 3.0) / 2.0)
    cs2 = (h * omk) ** 2
    return R ** p * torch.exp((1.0 / r - 1.0 / R) / cs2), omk * torch.sqrt((p + q) * (h / R) ** 2 + (1.0 + q) - q * R / r)


def _boxes(case):
    """The boxes' descriptions (as dust.Context takes them)."""
    g, sh = case["grid"], (case["shape"],) * 3
    if g == "boxes":
        return [dict(geom="cart", ndim=3, n=(n, n, n), bc_lo=("periodic",) * 3, bc_hi=("periodic",) * 3, shape=sh,
                     faces=[np.linspace(0.0, n / 64.0, n + 1)] * 3) for n in map(int, case["sizes"].split(","))]
    n = (case["n0"], case["n1"], case["n2"])
    if g == "square":
        return [dict(geom="cart", ndim=2, n=n, bc_lo=("periodic",) * 3, bc_hi=("periodic",) * 3, shape=sh,
                     faces=[np.linspace(0.0, 1.0, n[0] + 1), np.linspace(0.0, n[1] / n[0], n[1] + 1)])]
    if g in ("shear", "fargo"):
        w = 1.0 / n[0]
        bc = ("shear", "periodic", "periodic")
        return [dict(geom="cart", ndim=3, n=n, bc_lo=bc, bc_hi=bc, shape=sh,
                     faces=[np.linspace(-w * m, w * m, m + 1) for m in n])]
    if g == "cyl":
        bc = ("open", "periodic", "periodic")
        return [dict(geom="cyl", ndim=3, n=n, bc_lo=bc, bc_hi=bc, shape=sh,
                     faces=[0.4 * 6.25 ** (np.arange(n[0] + 1) / n[0]), np.linspace(0.0, TWO_PI, n[1] + 1),
                            np.linspace(-0.15, 0.15, n[2] + 1)])]
    bc = ("open", "open", "periodic")
    return [dict(geom="sph", ndim=3, n=n, bc_lo=bc, bc_hi=bc, shape=sh,
                 faces=[np.linspace(0.5, 5.0, n[0] + 1), np.linspace(math.pi / 2 - 0.3, math.pi / 2 + 0.3, n[1] + 1),
                        np.linspace(0.0, TWO_PI, n[2] + 1)])]


def _forces(case):
    g = case["grid"]
    if g in ("shear", "fargo"):
        return dict(kind="shearbox" if g == "shear" else "shearbox_fargo", **SHEAR)
    return dict(kind="pointmass", GM=1.0) if g in ("cyl", "sph") else dict(kind="none")


def _dt(case):
    """At most about one cell per step where the particles are fastest."""
    g = case["grid"]
    if g in ("boxes", "square"):
        return 0.01
    if g in ("shear", "fargo"):
        return 0.64 / case["n0"]
    phi = TWO_PI / (case["n1"] if g == "cyl" else case["n2"])
    return min(0.004, 0.9 * phi * (0.4 if g == "cyl" else 0.5) ** 1.5)


def _ghosted(f):
    return np.concatenate([[2 * f[0] - f[1]], f, [2 * f[-1] - f[-2]]])


def _inputs(case, seed):
    """Everything that a pass reads, on the GPU in the storage precision."""
    dev = "cuda"
    gen = torch.Generator(device=dev).manual_seed(int(seed) * 7919 + 17)
    rd = torch.float64 if case["prec"] == "f64" else torch.float32
    boxes, g = _boxes(case), case["grid"]

    def uni(*shape, lo=0.0, hi=1.0, dtype=torch.float64):
        return torch.rand(*shape, generator=gen, device=dev, dtype=dtype) * (hi - lo) + lo

    rho, vel, cells, spec, base = [], [[], [], []], [], [], 0
    nc = 2 if g == "square" else 3
    for b in boxes:
        nd, n = b["ndim"], b["n"]
        x = [torch.from_numpy(_ghosted(f)).to(dev) for f in b["faces"]]
        x = [0.5 * (f[1:] + f[:-1]) for f in x]
        shp = tuple(len(a) for a in reversed(x))
        X = [x[d].reshape([-1 if k == nd - 1 - d else 1 for k in range(nd)]).expand(shp) for d in range(nd)]
        noise = [1e-3 * torch.randn(shp, generator=gen, device=dev, dtype=torch.float64) for _ in range(nc + 1)]
        ph = uni(6, hi=TWO_PI).tolist()
        if g in ("cyl", "sph"):
            R, z = (X[0], X[2]) if g == "cyl" else (X[0] * torch.sin(X[1]), X[0] * torch.cos(X[1]))
            d, om = _disk(R, z)
            v = [torch.zeros(shp, device=dev, dtype=torch.float64) for _ in range(3)]
            v[1 if g == "cyl" else 2] = R * om
            rho.append(d * (1.0 + noise[nc]))
            v = [v[m] + noise[m] * R * om for m in range(3)]
        elif g in ("shear", "fargo"):
            k = TWO_PI / (b["faces"][0][-1] - b["faces"][0][0])
            rho.append(1.0 + 0.01 * torch.cos(k * X[0] + ph[0]) + noise[nc])
            v = [noise[m].clone() for m in range(3)]
            if g == "shear":
                v[1] -= SHEAR["q"] * SHEAR["Omega"] * X[0]
        else:
            # a bulk motion and a solenoidal flow of one wave along each axis
            k = [TWO_PI / (f[-1] - f[0]) for f in b["faces"]]
            v = [0.02 / (m + 1) + 0.01 * torch.sin(k[(m + 1) % nd] * X[(m + 1) % nd] + ph[m]) + noise[m]
                 for m in range(nd)]
            rho.append(1.0 + noise[nc])
        for m in range(nc):
            vel[m].append(v[m].reshape(-1))
        nact = int(np.prod(n[:nd]))
        if g == "boxes":
            # U{1..m} particles per cell and species, cell by cell
            most = max(1, int(case["ppc"]) // 2 - 1)
            cnt = torch.randint(1, most + 1, (nact * 4,), generator=gen, device=dev)
            # (the same total for every seed: one more or one less in some)
            miss = nact * 2 * (1 + most) - int(cnt.sum())
            some = (cnt < most if miss > 0 else cnt > 1).nonzero().view(-1)
            some = some[torch.randperm(some.numel(), generator=gen, device=dev)[:abs(miss)]]
            cnt[some] += 1 if miss > 0 else -1
            k4 = torch.repeat_interleave(torch.arange(nact * 4, device=dev, dtype=torch.int32), cnt)
            cells.append(k4 // 4 + base)
            spec.append((k4 % 4).to(torch.uint8))
        elif g == "cyl":
            # uniform in R, phi, z
            m = nact * int(case["ppc"])
            f = torch.from_numpy(b["faces"][0]).to(dev)
            i = (torch.searchsorted(f, uni(m, lo=0.4, hi=2.5), right=True) - 1).clamp_(0, n[0] - 1)
            rest = torch.randint(0, n[1] * n[2], (m,), generator=gen, device=dev)
            cells.append((i + n[0] * rest).to(torch.int32))
        else:
            cells.append(torch.randint(0, nact, (nact * int(case["ppc"]),), generator=gen, device=dev,
                                       dtype=torch.int32))
        base += nact
    cell = torch.cat(cells)
    N, ndim = cell.numel(), boxes[0]["ndim"]
    off = [torch.rand(N, generator=gen, device=dev, dtype=rd) - 0.5 for _ in range(ndim)]
    mom = [torch.zeros(N, device=dev, dtype=rd) for _ in range(nc)]
    P = dict(cell=cell, off=off, mom=mom)
    if g in ("cyl", "sph", "shear"):
        n, f = boxes[0]["n"], [torch.from_numpy(a).to(dev) for a in boxes[0]["faces"]]
        idx = [cell.long() % n[0], (cell.long() // n[0]) % n[1], cell.long() // (n[0] * n[1])]
        x = [0.5 * (f[d][idx[d]] + f[d][idx[d] + 1]) + off[d].double() * (f[d][idx[d] + 1] - f[d][idx[d]])
             for d in range(3)]
        if g == "shear":
            mom[1].copy_(-SHEAR["q"] * SHEAR["Omega"] * x[0])
        else:
            R, z = (x[0], x[2]) if g == "cyl" else (x[0] * torch.sin(x[1]), x[0] * torch.cos(x[1]))
            mom[1 if g == "cyl" else 2].copy_(R * R * _disk(R, z)[1])
    sp = dict(species_tau=None, species_mass=None)
    if case["drag"] == "species":
        P["species"] = torch.cat(spec) if spec else torch.zeros(N, device=dev, dtype=torch.uint8)
        dv = float(np.prod([a[1] - a[0] for a in boxes[0]["faces"]]))
        if g == "boxes":
            most = max(1, int(case["ppc"]) // 2 - 1)
            sp = dict(species_tau=list(TAUS), species_mass=[0.25 * dv / (0.5 * (1 + most))] * 4)
        else:
            sp = dict(species_tau=[0.1], species_mass=[dv / int(case["ppc"])])
    else:
        lo, hi = dict(stokes=(1e-3, 10.0), tau=(1e-6, 1.0), epstein=(1e-3, 1.0))[case["drag"]]
        P["drag"] = torch.exp(uni(N, lo=math.log(lo), hi=math.log(hi))).to(rd)
        P["mass"] = torch.full((N,), 0.06 / N, device=dev, dtype=rd)
    F = dict(rho=torch.cat([r.reshape(-1) for r in rho]).to(rd), vel=[torch.cat(v).to(rd) for v in vel[:nc]])
    return boxes, P, F, sp


def _zeros(F, k):
    return [torch.zeros_like(F["rho"]) for _ in range(k)]


# ------------------------------------------------------------------ the pass

def prepare(case, seed):
    boxes, P, F, sp = _inputs(case, seed)
    nc = len(F["vel"])
    F["dep"] = _zeros(F, nc + 1)
    ctx = dust.Context(boxes, prec=case["prec"], drag_mode=case["drag"], **sp)
    if case["grid"] in ("cyl", "sph"):
        ctx.set_tile(4, 16, 4)
    if case["det"]:
        ctx.set_deterministic(True)
    s = dict(case=case, ctx=ctx, P=P, F=F, dt=_dt(case), t=0.0, f=_forces(case))
    n = P["cell"].numel()
    if case["call"] == "cycle":
        s["S"] = dict(F, dep=_zeros(F, nc + 1))
    elif case["call"] == "density":
        s["rho_d"] = _zeros(F, 1)[0]
    elif case["call"] == "stages":
        s["vg"] = [torch.zeros_like(P["mom"][0]) for _ in range(nc)]
        s["imp"] = [torch.zeros_like(P["mom"][0]) for _ in range(nc + 1)]
        s["perm"] = torch.empty(n, device="cuda", dtype=torch.int32)
    elif case["call"] == "source":
        # the order that a step leaves (a step of no length moves nothing)
        ctx.step(P, F, 0.0, dust.forces_t(**s["f"]), 1, dust.STEP_FUSED)
    return s


def _state(P):
    return {k: P[k] for k in ("cell", "off", "mom", "drag", "species") if k in P}


def run(s):
    case, ctx, P, F, dt = s["case"], s["ctx"], s["P"], s["F"], s["dt"]
    f = dust.forces_t(t=s["t"], **s["f"])
    flags = dust.STEP_DIAG | (dust.STEP_APPLY_FEEDBACK if case["feedback"] else 0)
    call = case["call"]
    if call == "step":
        ctx.step(P, F, dt, f, case["nsteps"], flags | dust.STEP_FUSED | dust.STEP_REBIN_EVERY(case["rebin"]))
        s["t"] += dt * case["nsteps"]
        return dict(P=_state(P), vel=F["vel"], dep=F["dep"])
    if call == "unfused":
        ctx.step(P, F, dt, f, case["nsteps"], flags)
        s["t"] += dt * case["nsteps"]
        return dict(P=_state(P), vel=F["vel"], dep=F["dep"])
    if call == "cycle":
        S = s["S"]
        for a in S["dep"]:
            a.zero_()
        ctx.fill_ghosts(S, f, s["t"])
        ctx.drag_source(P, S, dt, f)
        ctx.fold_ghosts(S, f, s["t"])
        ctx.step(P, F, dt, f, 1, flags | dust.STEP_FUSED | dust.STEP_REBIN_EVERY(1))
        s["t"] += dt
        return dict(source=S["dep"][:-1], P=_state(P), vel=F["vel"], dep=F["dep"])
    if call == "source":
        for a in F["dep"]:
            a.zero_()
        ctx.drag_source(P, F, dt, f)
        return dict(source=F["dep"][:-1])
    if call == "density":
        s["rho_d"].zero_()
        ctx.deposit_mass(P, s["rho_d"])
        return dict(rho_d=s["rho_d"])
    # the step composed of the stage calls, particles put in cell order first
    ctx.bin(P, "cell", perm=s["perm"], apply=True)
    for a in F["dep"]:
        a.zero_()
    ctx.fill_ghosts(F, f, s["t"] + 0.5 * dt)
    ctx.push_expmid(P, None, dt, f, dust.PHASE_DRIFT1)
    ctx.gather(P, F, None, s["vg"])
    ctx.push_expmid(P, s["vg"], dt, f, dust.PHASE_KICK, s["imp"])
    ctx.deposit(P, s["imp"], F)
    ctx.push_expmid(P, None, dt, f, dust.PHASE_DRIFT2)
    ctx.fold_ghosts(F, f, s["t"] + 0.5 * dt)
    if case["feedback"]:
        ctx.apply_feedback(F)
    s["t"] += dt
    return dict(P=_state(P), perm=s["perm"], vel=F["vel"], dep=F["dep"])


def work(case):
    rs = 8 if case["prec"] == "f64" else 4
    boxes = _boxes(case)
    nd = boxes[0]["ndim"]
    nc = 2 if nd == 2 else 3
    cells = sum(float(np.prod(b["n"][:nd])) for b in boxes)
    if case["grid"] == "boxes":
        parts = cells * 4 * 0.5 * (1 + max(1, int(case["ppc"]) // 2 - 1))
    else:
        parts = cells * int(case["ppc"])
    attr = 1.0 if case["drag"] == "species" else 2.0 * rs
    state = 4.0 + rs * (nd + nc)
    st = 3.0 ** nd
    step_b = parts * (2 * state + attr) + cells * rs * (1 + nc + (nc + 1) + (nc if case["feedback"] else 0))
    step_f = parts * (st * (2 * nc + 2 * (nc + 1) + 2) + 120)
    src_b = parts * (state + attr) + cells * rs * (2 * nc)
    src_f = parts * (st * (4 * nc + 2) + 60)
    call = case["call"]
    if call == "source":
        return dict(bytes=src_b, flops=src_f)
    if call == "density":
        return dict(bytes=parts * (4.0 + rs * nd + 1.0) + cells * rs, flops=parts * (st * 3 + 20))
    if call == "cycle":
        return dict(bytes=src_b + step_b, flops=src_f + step_f)
    return dict(bytes=step_b * case["nsteps"], flops=step_f * case["nsteps"])


# ------------------------------------------------------------------ the pass in 64 bits

class _Grid:
    """One box in FP64: axes with a ghost cell at each end, fields as stored."""

    def __init__(self, b, shape):
        self.b, self.nd, self.n, self.geom, self.shape = b, b["ndim"], b["n"], b["geom"], shape
        self.f = [torch.from_numpy(_ghosted(f)).to("cuda") for f in b["faces"]]
        self.c = [0.5 * (f[1:] + f[:-1]) for f in self.f]
        self.w = [f[1:] - f[:-1] for f in self.f]
        self.shp = tuple(len(c) for c in reversed(self.c))
        iv = []
        for d, f in enumerate(self.f):
            a, e = f[:-1], f[1:]
            if self.geom == "cyl" and d == 0:
                v = 0.5 * (e * e - a * a)
            elif self.geom == "sph" and d == 0:
                v = (e ** 3 - a ** 3) / 3.0
            elif self.geom == "sph" and d == 1:
                v = torch.cos(a) - torch.cos(e)
            else:
                v = e - a
            iv.append(1.0 / v)
        self.iv = iv
        self.lo = [float(f[0]) for f in b["faces"]]
        self.hi = [float(f[-1]) for f in b["faces"]]
        self.shear = b["bc_lo"][0] == "shear"

    def ax(self, a, d, s):
        """Index of array a (stored order) along axis d."""
        return a.select(self.nd - 1 - d, s)

    def locate(self, x, d):
        i = torch.searchsorted(self.f[d][1:-1].contiguous(), x, right=True) - 1
        return i.clamp_(0, self.n[d] - 1)

    def weights(self, x, i, d):
        c, w = self.c[d][i + 1], self.w[d][i + 1]
        e = (x - c) / w
        tsc = self.shape == "tsc"
        zero = torch.zeros_like(e)
        m, p = 0.5 - e, 0.5 + e
        if self.geom == "cyl" and d == 0:
            nu = c / w
            if tsc:
                den = 3 * (e + nu)
                lo, hi = (e + 3 * nu - 2) / den * 0.5 * m * m, (e + 3 * nu + 2) / den * 0.5 * p * p
            else:
                den = 2 * (e + nu)
                lo, hi = (e + 2 * nu - 1) / den * (-e), (e + 2 * nu + 1) / den * e
        elif self.geom == "sph" and d == 0:
            nu = c / w
            if tsc:
                den = 6 * (e + nu) ** 2 + 1
                lo = (e * e + (4 * nu - 3) * e + 6 * nu * nu - 8 * nu + 2.75) / den * 0.5 * m * m
                hi = (e * e + (4 * nu + 3) * e + 6 * nu * nu + 8 * nu + 2.75) / den * 0.5 * p * p
            else:
                den = 12 * (e + nu) ** 2 + 1
                lo = ((2 * e + 3 * nu - 1.5) ** 2 + 3 * (nu - 0.5) ** 2) / den * (-e)
                hi = ((2 * e + 3 * nu + 1.5) ** 2 + 3 * (nu + 0.5) ** 2) / den * e
        elif self.geom == "sph" and d == 1:
            # the shape's share beyond each face, with the metric sin(theta)
            sp, sh = torch.sin(x), torch.sin(0.5 * w)
            if tsc:
                den = 4 * sp * sh * sh
                hp, hm = p * w, m * w
                a, b = c + 0.5 * w, c - 0.5 * w
                series = [1.0 / 6, -1.0 / 120, 1.0 / 5040, -1.0 / 362880]
                hs = [sum(k * h ** (3 + 2 * q) for q, k in enumerate(series)) for h in (hp, hm)]
                hi = (torch.cos(a) * hs[0] + 2 * torch.sin(a) * torch.sin(0.5 * hp) ** 2) / den
                lo = (-torch.cos(b) * hs[1] + 2 * torch.sin(b) * torch.sin(0.5 * hm) ** 2) / den
            else:
                hi = torch.sin(c + 0.5 * w + 0.5 * e * w) * torch.sin(0.5 * e * w) / (sp * sh)
                lo = torch.sin(c - 0.5 * w + 0.5 * e * w) * torch.sin(-0.5 * e * w) / (sp * sh)
        elif tsc:
            lo, hi = 0.5 * m * m, 0.5 * p * p
        else:
            lo, hi = -e, e
        if not tsc:
            lo, hi = torch.where(e < 0, lo, zero), torch.where(e > 0, hi, zero)
        return [lo, 1.0 - lo - hi, hi]

    def stencil(self, x, idx):
        """(stored index, weight) of each cell of the stencil, one at a time."""
        w = [self.weights(x[d], idx[d], d) for d in range(self.nd)]
        g0, g1 = self.shp[-1], self.shp[-2]
        for c in range(3 if self.nd > 2 else 1):
            for b in range(3):
                for a in range(3):
                    s = (idx[0] + a) + g0 * (idx[1] + b)
                    wt = w[0][a] * w[1][b]
                    iv = self.iv[0][idx[0] + a] * self.iv[1][idx[1] + b]
                    if self.nd > 2:
                        s = s + g0 * g1 * (idx[2] + c)
                        wt = wt * w[2][c]
                        iv = iv * self.iv[2][idx[2] + c]
                    yield s, wt, iv

    def shift(self, t):
        u = SHEAR["q"] * SHEAR["Omega"] * (self.hi[0] - self.lo[0])
        s = (u * t / ((self.hi[1] - self.lo[1]) / self.n[1])) % self.n[1]
        return u, s

    def rows(self, a, s):
        """Rows of a (.., y) taken at j + s, linear between two cells."""
        k, fr = int(math.floor(s)), s - math.floor(s)
        return (1 - fr) * torch.roll(a, -k, -1) + fr * torch.roll(a, -k - 1, -1)

    def fill(self, arrs, vy, t, boost):
        for k, a in enumerate(arrs):
            if self.shear:
                u, s = self.shift(t)
                u = u if boost and k == vy else 0.0
                act = a[1:-1, 1:-1]
                a[1:-1, 1:-1, -1] = self.rows(act[:, :, 1], s) - u
                a[1:-1, 1:-1, 0] = self.rows(act[:, :, -2], -s) + u
            for d in range(1 if self.shear else 0, self.nd):
                if self.b["bc_lo"][d] == "periodic":
                    self.ax(a, d, 0).copy_(self.ax(a, d, self.n[d]))
                    self.ax(a, d, self.n[d] + 1).copy_(self.ax(a, d, 1))

    def fold(self, arrs, t, boost):
        def onto(a, d):
            self.ax(a, d, self.n[d]).add_(self.ax(a, d, 0))
            self.ax(a, d, 1).add_(self.ax(a, d, self.n[d] + 1))
            self.ax(a, d, 0).zero_()
            self.ax(a, d, self.n[d] + 1).zero_()

        for a in arrs:
            for d in range(self.nd - 1, 0 if self.shear else -1, -1):
                if self.b["bc_lo"][d] == "periodic":
                    onto(a, d)
        if self.shear:
            u, s = self.shift(t)
            dy = arrs[1].clone()
            for k, a in enumerate(arrs):
                right, left = a[1:-1, 1:-1, -1].clone(), a[1:-1, 1:-1, 0].clone()
                if boost and k == 3:
                    right += u * dy[1:-1, 1:-1, -1]
                    left -= u * dy[1:-1, 1:-1, 0]
                a[1:-1, 1:-1, 1] += self.rows(right, -s)
                a[1:-1, 1:-1, -2] += self.rows(left, s)
                a[:, :, 0].zero_()
                a[:, :, -1].zero_()

    def scale(self, x):
        one = torch.ones_like(x[0])
        if self.geom == "cyl":
            return [one, x[0], one]
        if self.geom == "sph":
            return [one, x[0], x[0] * torch.sin(x[1])]
        return [one] * self.nd


class _Set:
    """The particles of one box in FP64 coordinates."""

    def __init__(self, g, P, base, sel, sp, drag):
        self.g = g
        c = P["cell"][sel].long() - base
        i = [c % g.n[0], (c // g.n[0]) % g.n[1], c // (g.n[0] * g.n[1])][: g.nd]
        self.x = [g.c[d][i[d] + 1] + P["off"][d][sel].double() * g.w[d][i[d] + 1] for d in range(g.nd)]
        self.p = [m[sel].double() for m in P["mom"]]
        self.i = i
        self.live = torch.ones_like(c, dtype=torch.bool)
        if drag == "species":
            k = P["species"][sel].long()
            self.m = torch.tensor(sp["species_mass"], device="cuda", dtype=torch.float64)[k]
            self.tau = torch.tensor(sp["species_tau"], device="cuda", dtype=torch.float64)[k]
        else:
            self.m, self.tau = P["mass"][sel].double(), P["drag"][sel].double()

    def inverse_tau(self, drag, rho=None):
        if drag == "stokes":
            R = self.x[0]
            return R ** -1.5 / self.tau
        return rho / self.tau if drag == "epstein" else 1.0 / self.tau

    def bounds(self, t, fargo):
        g = self.g
        for d in range(g.nd):
            L = g.hi[d] - g.lo[d]
            x = self.x[d]
            if d == 0 and g.shear:
                k = torch.floor((x - g.lo[0]) / L)
                u, s = g.shift(t)
                self.x[0] = x - k * L
                self.x[1] = self.x[1] + k * s * (g.hi[1] - g.lo[1]) / g.n[1]
                if not fargo:
                    self.p[1] = self.p[1] + k * u
            elif g.b["bc_lo"][d] == "periodic":
                self.x[d] = g.lo[d] + torch.remainder(x - g.lo[d], L)
            else:
                self.live &= (x >= g.lo[d]) & (x < g.hi[d])
                self.x[d] = x.clamp(g.lo[d], g.hi[d])
        self.i = [g.locate(self.x[d], d) for d in range(g.nd)]

    def drift(self, h, first, t, fargo):
        x, p, g = self.x, self.p, self.g
        if g.geom == "cart":
            qO = SHEAR["q"] * SHEAR["Omega"] if fargo else 0.0
            if first or not fargo:
                x[0] = x[0] + h * p[0]
            x[1] = x[1] + h * (p[1] - qO * x[0])
            if fargo and not first:
                x[0] = x[0] + h * p[0]
            if g.nd > 2:
                x[2] = x[2] + h * p[2]
        elif g.geom == "cyl":
            if first:
                x[0] = x[0] + h * p[0]
            x[1] = x[1] + h * p[1] / x[0] ** 2
            if not first:
                x[0] = x[0] + h * p[0]
            x[2] = x[2] + h * p[2]
        elif first:
            x[0] = x[0] + h * p[0]
            x[1] = x[1] + h * p[1] / x[0] ** 2
            x[2] = x[2] + h * p[2] / (x[0] * torch.sin(x[1])) ** 2
        else:
            x[2] = x[2] + h * p[2] / (x[0] * torch.sin(x[1])) ** 2
            x[1] = x[1] + h * p[1] / x[0] ** 2
            x[0] = x[0] + h * p[0]
        self.bounds(t, fargo)

    def gather(self, rho, vel):
        """Gas density and the slip of each canonical component."""
        g, sc = self.g, self.g.scale(self.x)
        u = [self.p[m] / sc[m] for m in range(len(vel))]
        r, v = None, [torch.zeros_like(self.x[0]) for _ in vel]
        if rho is not None:
            r = torch.zeros_like(self.x[0])
        for s, w, _ in g.stencil(self.x, self.i):
            if r is not None:
                r += w * rho.view(-1)[s]
            for m, a in enumerate(vel):
                v[m] += w * (a.view(-1)[s] - u[m])
        return r, [v[m] * sc[m] for m in range(len(vel))]

    def kick(self, dt, it, sl, kind):
        p, g = self.p, self.g
        h = dt * it
        c = -torch.expm1(-h)
        small = h < 1e-3
        psi = torch.where(small, -h / 2 * (1 - h / 3 * (1 - h / 4 * (1 - h / 5))), c / torch.where(small, 1.0, h) - 1.0)
        h1 = dt * (1 + psi)
        zero = torch.zeros_like(c)
        n = len(p)
        if kind in ("shearbox", "shearbox_fargo"):
            Om, q = SHEAR["Omega"], SHEAR["q"]
            if kind == "shearbox":
                an = [2 * Om * (p[1] + q * Om * self.x[0]), -2 * Om * p[0], zero]
                W2, k = Om * h1, -Om
            else:
                an = [2 * Om * p[1], (q - 2) * Om * p[0], zero]
                W2, k = Om * h1 * (1 - 0.5 * q), 0.5 * (q - 2) * Om
            W1 = Om * h1
            r = [c * sl[d] + h1 * an[d] for d in range(3)]
            den = 1 / (1 + W1 * W2)
            dp = [(r[0] + W1 * r[1]) * den, (r[1] - W2 * r[0]) * den, r[2]]
            a = [an[0] + Om * dp[1], an[1] + k * dp[0], zero]
        elif g.geom == "cyl":
            R, z = self.x[0], self.x[2]
            r3 = (R * R + z * z) ** 1.5
            d1 = c * sl[1]
            a = [0.5 * (p[1] ** 2 + (p[1] + d1) ** 2) / R ** 3 - R / r3, zero, -z / r3]
            dp = [c * sl[d] + h1 * a[d] for d in range(3)]
        elif g.geom == "sph":
            r, st, ct = self.x[0], torch.sin(self.x[1]), torch.cos(self.x[1])
            lp = 0.5 * (p[2] ** 2 + (p[2] + c * sl[2]) ** 2)
            a1 = lp * ct / (r * r * st ** 3)
            lt = 0.5 * (p[1] ** 2 + (p[1] + c * sl[1] + h1 * a1) ** 2)
            a = [lt / r ** 3 + lp / (r ** 3 * st * st) - 1 / (r * r), a1, zero]
            dp = [c * sl[d] + h1 * a[d] for d in range(3)]
        else:
            a, dp = [zero] * n, [c * sl[d] for d in range(n)]
        sc = g.scale(self.x)
        J = [self.m * (c * sl[d] + dt * psi * a[d]) for d in range(n)]
        J.append(sum((p[d] + 0.5 * dp[d]) / sc[d] * J[d] / sc[d] for d in range(n)))
        self.p = [p[d] + dp[d] for d in range(n)]
        return J

    def deposit(self, dep, q, sgn):
        q = [torch.where(self.live, a, torch.zeros_like(a)) for a in q]
        for s, w, iv in self.g.stencil(self.x, self.i):
            for m in range(len(q)):
                dep[m].view(-1).index_add_(0, s, sgn * w * iv * q[m])


def exact(case, seed):
    boxes, P, F, sp = _inputs(case, seed)
    call, drag, dt, f = case["call"], case["drag"], _dt(case), _forces(case)
    fargo = f["kind"] == "shearbox_fargo"
    boost = f["kind"] == "shearbox"
    nc, n = len(F["vel"]), P["cell"].numel()
    if n * case["nsteps"] > 1.5e9:
        return None
    out = {k: [torch.zeros(F["rho"].numel(), device="cuda", dtype=torch.float64) for _ in range(nc + 1)]
           for k in ("vel", "dep", "source")}
    parts = dict(off=[torch.zeros(n, device="cuda", dtype=torch.float64) for _ in range(boxes[0]["ndim"])],
                 mom=[torch.zeros(n, device="cuda", dtype=torch.float64) for _ in range(nc)])
    order = torch.sort(P["cell"], stable=True)[1] if call == "stages" else None
    base = at = 0
    for b in boxes:
        g = _Grid(b, case["shape"])
        nact, nst = int(np.prod(b["n"][: g.nd])), int(np.prod(g.shp))
        sel = ((P["cell"] >= base) & (P["cell"] < base + nact)).nonzero().view(-1) if order is None else order
        if order is None and case["grid"] == "boxes":
            # (neighbours in memory are of one cell here, where the sums below would queue)
            sel = sel[torch.randperm(sel.numel(), device="cuda")]
        gas = lambda a: a[at:at + nst].double().view(g.shp).clone()  # noqa: E731
        rho, vel = gas(F["rho"]), [gas(v) for v in F["vel"]]
        dep = [torch.zeros_like(rho) for _ in range(nc + 1)]
        s = _Set(g, P, base, sel, sp, drag)
        if call == "density":
            s.deposit(dep, [s.m], 1.0)
            out["dep"][0][at:at + nst] = dep[0].view(-1)
        if call in ("source", "cycle"):
            src = [torch.zeros_like(rho) for _ in range(nc + 1)]
            v0 = [a.clone() for a in vel]
            # (a source alone: the step of no length before it fills the ghosts)
            g.fill(v0, 1, 0.0, boost)
            k = torch.clamp(s.inverse_tau(drag), max=1.0 / dt) * s.m
            s.deposit(src, [k * a for a in s.gather(None, v0)[1]], -1.0)
            if call == "cycle":
                g.fold(src, 0.0, boost)
            for m in range(nc):
                out["source"][m][at:at + nst] = src[m].view(-1)
        if call in ("step", "unfused", "cycle", "stages"):
            t = 0.0
            for _ in range(case["nsteps"]):
                for a in dep:
                    a.zero_()
                g.fill([rho] + vel, 2, t + 0.5 * dt, boost)
                s.drift(0.5 * dt, True, t + 0.5 * dt, fargo)
                r, sl = s.gather(rho if drag == "epstein" else None, vel)
                J = s.kick(dt, s.inverse_tau(drag, r), sl, f["kind"])
                s.deposit(dep, J, -1.0)
                s.drift(0.5 * dt, False, t + dt, fargo)
                g.fold(dep, t + 0.5 * dt, boost)
                if case["feedback"]:
                    act = (slice(1, -1),) * g.nd
                    R = g.c[0][1:-1]
                    for m in range(nc):
                        q = dep[m][act] / rho[act]
                        if g.geom != "cart" and m == 1:
                            q = q / R
                        if g.geom == "sph" and m == 2:
                            q = q / (R * torch.sin(g.c[1][1:-1])[:, None])
                        vel[m][act] += q
                t += dt
            for m in range(nc + 1):
                out["dep"][m][at:at + nst] = dep[m].view(-1)
            for m in range(nc):
                out["vel"][m][at:at + nst] = vel[m].view(-1)
                to = sel if order is None else slice(None)
                parts["mom"][m][to] = s.p[m]
            for d in range(g.nd):
                parts["off"][d][sel if order is None else slice(None)] = \
                    (s.x[d] - g.c[d][s.i[d] + 1]) / g.w[d][s.i[d] + 1]
        base, at = base + nact, at + nst
    if call == "density":
        return dict(rho_d=out["dep"][0])
    if call == "source":
        return dict(source=out["source"][:nc])
    # the fused step reorders the particles by its own tiles: no value by slot
    own = dict(parts) if call in ("unfused", "stages") and int(not (~s.live).any()) else None
    r = dict(P=own, vel=out["vel"][:nc], dep=out["dep"])
    if call == "cycle":
        r["source"] = out["source"][:nc]
    return r
