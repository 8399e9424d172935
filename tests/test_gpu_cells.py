"""The rebinning step on both sides of its lines against the oracle: a
particle per lane or a cell per thread (9, 28 and 56 particles per cell on the
FP32 uniform-Cartesian, other Cartesian and curvilinear paths), few tiles
shared by several workgroups, tiles cut by the box, axes thinner than a tile,
open faces, CIC and mixed shapes, particles without a cell, crowded cells.
Tolerances: those of the parity tests (FP32 1e-5, FP64 1e-12)."""
import dataclasses

import numpy as np
import pytest

from gpu_common import compare_step, download, workload_from_state
from oracle.run import OracleRun
from paper_1908_10793_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _with_ppc(w, ppc, seed=9):
    """w with ppc particles per cell on average, drawn from its own, at
    uniform random offsets; every 97th without a cell, one cell crowded."""
    r = np.random.default_rng(seed)
    _, ncell = w.cell_bases()
    n = int(ncell * ppc)
    idx = np.sort(r.integers(0, w.n, size=n))[r.permutation(n)]
    nd = w.boxes[0]["ndim"]
    off = np.zeros((n, 3), dtype=w.np_dtype)
    off[:, :nd] = np.clip((r.random((n, nd)) - 0.5).astype(w.np_dtype), -0.5, 0.4999)
    cell = w.cell[idx].copy()
    cell[: n // 50] = cell[0]
    cell[5::97] = -1
    pick = {k: getattr(w, k)[idx] for k in ("drag", "mass", "species") if getattr(w, k) is not None}
    return dataclasses.replace(w, cell=cell, off=off, mom=w.mom[idx], **pick)


def _box(dtype, shape, bc, n=(19, 9, 6)):
    w = synth.batched_boxes(sizes=(max(n),), max_per_species=2, dt=0.05, dtype=dtype)
    b = dict(w.boxes[0], n=n, bc_lo=bc, bc_hi=bc, shape=shape, faces=[w.boxes[0]["faces"][d][:n[d] + 1] for d in range(3)])
    g = w.gas[0]
    cut = tuple(slice(0, n[d] + 2) for d in (2, 1, 0))
    cell = np.arange(w.n, dtype=np.int32) % int(np.prod(n))
    return dataclasses.replace(w, boxes=[b], cell=cell,
                               gas=[dict(rho=g["rho"][cut].copy(), vel=[v[cut].copy() for v in g["vel"]])])


def _workload(name, dtype):
    if name == "shear":
        return synth.shearing_box(n=(18, 11, 7), dt=0.05, dtype=dtype)
    if name == "fargo":
        return synth.shearing_box(n=(10, 9, 5), dt=0.05, dtype=dtype, fargo=True)
    if name == "thin":
        return synth.shearing_box(n=(35, 3, 2), dt=0.05, dtype=dtype)
    if name == "boxes":
        return synth.batched_boxes(sizes=(3, 9, 12), max_per_species=4, dt=0.05, dtype=dtype)
    if name == "open_mixed":
        # (ghosts of an open face beside a periodic one are images only along the
        # later axis)
        return _box(dtype, ("tsc", "cic", "tsc"), ("open", "open", "periodic"))
    if name == "cic":
        return _box(dtype, ("cic",) * 3, ("periodic",) * 3)
    if name == "square":
        return synth.cart2d_periodic(n=(33, 21), shape="tsc", dtype=dtype)
    if name == "cyl":
        return synth.cylindrical_disk(n=(13, 17, 6), npart=5000, dt=0.02, dtype=dtype)
    return synth.spherical_disk(n=(13, 9, 11), ppc=2, dt=0.02, dtype=dtype)


CART = [(n, d, p) for n in ("shear", "thin", "boxes", "open_mixed", "cic") for d, p in (("f32", 4), ("f32", 9), ("f32", 11),
                                                                                        ("f64", 3), ("f64", 30))]
OTHER = [("fargo", "f32", 12), ("fargo", "f32", 29), ("fargo", "f64", 12), ("square", "f32", 20), ("square", "f64", 31),
         ("cyl", "f32", 5), ("cyl", "f32", 40), ("cyl", "f32", 58), ("cyl", "f64", 7), ("sph", "f32", 3), ("sph", "f32", 50),
         ("sph", "f64", 60)]


@pytest.mark.parametrize("name,dtype,ppc", CART + OTHER)
def test_rebinning_step_matches_oracle(name, dtype, ppc):
    from paper_1908_10793_amd import dust
    w = _with_ppc(_workload(name, dtype), ppc)
    print(f"[cells] {name} {dtype} {ppc} n={w.n}", flush=True)
    ctx = dust.context_for(w)
    P, F = dust.upload(w, ctx)
    flags = dust.STEP_DIAG | dust.STEP_FUSED | (dust.STEP_APPLY_FEEDBACK if w.apply_feedback else 0)
    t = w.t0
    for s in range(2):
        st_in = download(ctx, P, F, w)
        before = ctx.status()
        ctx.step(P, F, w.dt, dust.forces_for(w, t), 1, flags)
        st_out = download(ctx, P, F, w)
        diag = ctx.status()
        wi = workload_from_state(w, st_in, t)
        run = OracleRun(wi)
        run.step(1)
        # (gas that the heavy feedback of so many particles changes is not compared)
        compare_step(dataclasses.replace(wi, apply_feedback=False), st_in, st_out, run, w.dtype, label=f"{name} {s}")
        d = {k: np.asarray(diag[k]) for k in ("p_part", "p_grid", "sum_abs_j")}
        res = np.abs(d["p_part"] + d["p_grid"]).max() / max(float(d["sum_abs_j"]), 1e-300)
        assert res < (1e-12 if dtype == "f64" else 2e-6), res
        assert diag["n_removed"] - before["n_removed"] == int((st_in["cell"] >= 0).sum() - (st_out["cell"] >= 0).sum())
        t += w.dt
