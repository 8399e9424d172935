"""Ghost fill, fold and feedback where the sets of ghost cells are smallest or
mixed: axes of one and two cells, open next to periodic faces, several boxes
of a launch and more than one launch holds, against the oracle.

The fill copies values or interpolates two (FP64), the fold adds at most 27
values of a cell, the feedback divides once: in FP64 errors of some 30 ulp of
the largest value (1e-13 of it), in FP32 of 30 * 2^-24 (2e-6).
"""
import numpy as np
import pytest

import oracle as O
from oracle.run import make_box, make_forces

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

PER, OPEN, SHEAR = "periodic", "open", "shear"
SETS = {
    "square": [((1, 5), (PER, PER)), ((4, 1), (PER, PER)), ((3, 7), (OPEN, PER)), ((5, 2), (PER, OPEN)),
               ((2, 3), (OPEN, OPEN))],
    "box": [((1, 1, 1), (PER, PER, PER)), ((2, 3, 1), (PER, PER, PER)), ((5, 4, 3), (PER, OPEN, PER)),
            ((5, 4, 3), (OPEN, PER, OPEN)), ((3, 2, 9), (PER, PER, OPEN)), ((7, 1, 2), (OPEN, OPEN, PER))],
    "shear": [((1, 6, 3), (SHEAR, PER, PER)), ((5, 1, 2), (SHEAR, PER, OPEN)), ((9, 8, 7), (SHEAR, PER, PER)),
              ((4, 3, 5), (PER, PER, PER))],
    "many": [((3 + k % 4, 2 + k % 3, 4), (PER, PER, PER) if k % 2 else (OPEN, PER, OPEN)) for k in range(37)],
}


def _box(n, bc):
    nd = len(n)
    bc = tuple(bc) + (PER,) * (3 - nd)
    faces = [np.linspace(0.0, 0.5 * n[d], n[d] + 1) for d in range(nd)]
    return dict(geom="cart", ndim=nd, n=tuple(n) + (1,) * (3 - nd), bc_lo=bc, bc_hi=bc, shape=("cic",) * 3, faces=faces)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("name", list(SETS))
def test_fill_fold_and_feedback_match_oracle(name, dtype):
    from paper_1908_10793_amd import dust
    boxes = [_box(n, bc) for n, bc in SETS[name]]
    nd = boxes[0]["ndim"]
    fd = dict(kind="shearbox", Omega=1.0, q=1.5) if name == "shear" else dict(kind="none")
    print(f"[grid edges] {name} {dtype}", flush=True)
    ctx = dust.Context(boxes, prec=dtype)
    fr = dust.forces_t(**fd)
    ob, of = [make_box(b) for b in boxes], make_forces(fd)
    rng = np.random.default_rng(3)
    shapes = [b.ghosted_shape for b in ob]
    rd = ctx.real_dtype
    npd = np.float64 if dtype == "f64" else np.float32
    tol = 1e-13 if dtype == "f64" else 2e-6

    def rand(lo):
        return [(lo + rng.random(s)).astype(npd).astype(np.float64) for s in shapes]

    def up(parts):
        return torch.from_numpy(np.concatenate([x.ravel() for x in parts])).to("cuda", rd)

    def close(t, parts, what):
        ref = np.concatenate([x.ravel() for x in parts])
        err = np.abs(t.cpu().numpy().astype(np.float64) - ref).max()
        assert err <= tol * max(1.0, np.abs(ref).max()), (what, err)

    for t in (0.0, 0.37, 3.9):
        rho, vel, dep = rand(1.0), [rand(-0.5) for _ in range(nd)], [rand(-0.5) for _ in range(nd + 1)]
        F = {"rho": up(rho), "vel": [up(v) for v in vel], "dep": [up(d) for d in dep]}
        fo = [O.Fields(b, rho[e].copy(), [v[e].copy() for v in vel], dep=[d[e].copy() for d in dep])
              for e, b in enumerate(ob)]
        ctx.fill_ghosts(F, fr, t)
        for b, f in zip(ob, fo):
            O.fill_ghosts(b, of, t, f)
        close(F["rho"], [f.rho for f in fo], "rho")
        for c in range(nd):
            close(F["vel"][c], [f.vel[c] for f in fo], f"vel {c}")
        ctx.fold_ghosts(F, fr, t)
        for b, f in zip(ob, fo):
            O.fold_ghosts(b, of, t, f)
        for c in range(nd + 1):
            close(F["dep"][c], [f.dep[c] for f in fo], f"dep {c}")
        ctx.apply_feedback(F)
        act = (Ellipsis,) + (slice(1, -1),) * nd
        for f in fo:
            for c in range(nd):
                f.vel[c][act] += f.dep[c][act] / f.rho[act]
        for c in range(nd):
            close(F["vel"][c], [f.vel[c] for f in fo], f"feedback {c}")


@pytest.mark.parametrize("name", list(SETS))
def test_step_without_particles_fills_folds_and_counts(name):
    """A step whose particles have no cell: ghosts filled, deposits cleared,
    the time advanced and the steps counted, also with many boxes."""
    from paper_1908_10793_amd import dust
    boxes = [_box(n, bc) for n, bc in SETS[name]]
    nd = boxes[0]["ndim"]
    fd = dict(kind="shearbox", Omega=1.0, q=1.5) if name == "shear" else dict(kind="none")
    ctx = dust.Context(boxes, prec="f64", drag_mode="species", species_tau=[1.0], species_mass=[1.0])
    fr = dust.forces_t(**fd)
    ob, of = [make_box(b) for b in boxes], make_forces(fd)
    rng = np.random.default_rng(4)
    tot = sum(int(np.prod(b.ghosted_shape)) for b in ob)
    vel = rng.random((nd, tot))
    F = {"rho": torch.ones(tot, dtype=torch.float64, device="cuda"),
         "vel": [torch.from_numpy(v).cuda() for v in vel],
         "dep": [torch.full((tot,), 7.0, dtype=torch.float64, device="cuda") for _ in range(nd + 1)]}
    n = 1000
    P = {"cell": torch.full((n,), -1, dtype=torch.int32, device="cuda"),
         "off": [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(nd)],
         "mom": [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(nd)]}
    dt = 0.125
    for flags in (dust.STEP_DIAG, dust.STEP_DIAG | dust.STEP_FUSED):
        ctx.step(P, F, dt, fr, 3, flags | dust.STEP_APPLY_FEEDBACK)
        assert all(float(d.abs().max()) == 0.0 for d in F["dep"])
        at = 0
        for e, b in enumerate(ob):
            size = int(np.prod(b.ghosted_shape))
            g = [v[at:at + size].reshape(b.ghosted_shape).copy() for v in vel]
            f = O.Fields(b, np.ones(b.ghosted_shape), g, dep=[np.zeros(b.ghosted_shape) for _ in range(nd + 1)])
            O.fill_ghosts(b, of, 2.5 * dt, f)   # the fill of the last step, at its midpoint
            for c in range(nd):
                got = F["vel"][c][at:at + size].cpu().numpy().reshape(b.ghosted_shape)
                assert np.abs(got - f.vel[c]).max() <= 1e-13 * max(1.0, np.abs(f.vel[c]).max()), (e, c)
            at += size
    assert ctx.status()["steps"] == 6
