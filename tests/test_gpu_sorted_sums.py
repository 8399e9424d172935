"""The particle-to-grid sums over sorted particles (deposit stage, drag
source, dust density) against the same calls on slices of the particles.

A call of 4096 particles or more, with a quarter per cell or more, sorts the
particles and sums them tile by tile; a slice below that size adds particle
by particle.  Both are the same sums, so the whole call must equal the sum of
its slices.  Tolerances (normwise, per channel): FP64 contributions and sums
round at 2^-53, some 1e3 of them per word: 1e-12; FP32 sums of up to some 1e3
contributions of one sign: 1e-5, the bar of the parity tests.  (The unfused
step takes this path in the parity tests, which compare it with the oracle.)
"""
import numpy as np
import pytest

from paper_1908_10793_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SLICE = 4000   # below the sorted path's smallest call


def _workload(name, dtype):
    kw = dict(dtype=dtype)
    if name == "square_ragged":      # 2-D tiles with remainders on both axes
        return synth.cart2d_periodic(n=(33, 50), ppc=10, shape="cic", **kw)
    if name == "square_smallest":    # one tile
        return synth.cart2d_periodic(n=(16, 16), ppc=64, shape="tsc", **kw)
    if name == "box_thin":           # fewer cells than a tile along two axes
        return synth.shearing_box(n=(700, 3, 2), **kw)
    if name == "box_ragged":
        return synth.shearing_box(n=(17, 13, 11), **kw)
    if name == "boxes":              # several boxes, one smaller than a tile
        return synth.batched_boxes(sizes=(3, 9, 12), max_per_species=5, **kw)
    if name == "cells_crowded":      # one cell holds a workgroup's slots and more
        w = synth.batched_boxes(sizes=(8,), max_per_species=16, **kw)
        w.cell[: w.n // 2] = 77
        return w
    if name == "disk":
        return synth.cylindrical_disk(n=(19, 23, 7), npart=20011, **kw)
    return synth.spherical_disk(n=(13, 21, 17), ppc=4, **kw)


NAMES = ["square_ragged", "square_smallest", "box_thin", "box_ragged", "boxes", "cells_crowded", "disk", "sphere"]


def _slices(P, n):
    for a in range(0, n, SLICE):
        sl = slice(a, min(n, a + SLICE))
        yield {k: ([t[sl].contiguous() for t in v] if isinstance(v, list) else v[sl].contiguous())
               for k, v in P.items()}, sl


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("name", NAMES)
def test_sorted_sums_equal_the_sums_of_slices(name, dtype):
    from paper_1908_10793_amd import dust
    w = _workload(name, dtype)
    print(f"[sorted sums] {name} {dtype} n={w.n}", flush=True)
    assert w.n >= 16384
    ctx = dust.context_for(w)
    P, F = dust.upload(w, ctx)
    g = torch.Generator(device="cuda").manual_seed(5)
    order = torch.randperm(w.n, generator=g, device="cuda")
    P = {k: ([t[order].contiguous() for t in v] if isinstance(v, list) else v[order].contiguous())
         for k, v in P.items()}
    P["cell"][5::97] = -1   # particles without a cell
    rd = ctx.real_dtype
    P["mom"] = [m + 0.01 * torch.rand(w.n, generator=g, device="cuda", dtype=rd) for m in P["mom"]]
    fr = dust.forces_for(w, 0.0)
    ctx.fill_ghosts(F, fr, 0.0)
    imp = [torch.rand(w.n, generator=g, device="cuda", dtype=rd) for _ in F["dep"]]
    tol = 1e-12 if dtype == "f64" else 1e-5

    def compare(call, what):
        whole = [torch.zeros_like(d) for d in F["dep"]]
        parts = [torch.zeros_like(d) for d in F["dep"]]
        call(P, imp, dict(F, dep=whole))
        flags = ctx.status()["flag_names"]
        for Q, sl in _slices(P, w.n):
            call(Q, [q[sl].contiguous() for q in imp], dict(F, dep=parts))
        # (the thin box's displacements leave some offsets out of range)
        assert flags == ctx.status()["flag_names"], what
        for c, (a, b) in enumerate(zip(whole, parts)):
            a, b = a.double().cpu().numpy(), b.double().cpu().numpy()
            scale = np.abs(b).max()
            assert np.abs(a - b).max() <= tol * scale, (what, c, np.abs(a - b).max() / max(scale, 1e-300))

    compare(lambda Q, q, G: ctx.deposit(Q, q, G), "deposit")
    compare(lambda Q, q, G: ctx.drag_source(Q, G, w.dt, fr), "source")
    compare(lambda Q, q, G: ctx.deposit_mass(Q, G["dep"][0]), "density")


def test_sorted_sums_flag_what_the_particle_kernels_flag():
    """Cell ids and offsets out of range, a species beyond the table and a
    non-finite momentum raise their sticky bits on the sorted path too, and a
    particle without a valid cell adds nothing."""
    from paper_1908_10793_amd import dust
    w = _workload("box_ragged", "f32")
    ctx = dust.context_for(w)
    P, F = dust.upload(w, ctx)
    fr = dust.forces_for(w, 0.0)
    rho = torch.zeros_like(F["rho"])
    P["cell"][100] = 17 * 13 * 11
    ctx.deposit_mass(P, rho)
    assert ctx.status()["flag_names"] == ["bad_cell"]
    total = float(rho.double().sum()) * 8.0 / (17 * 13 * 11)   # (cells of a box of side 2)
    want = (w.n - 1) * w.species_mass[0]
    assert abs(total - want) <= 1e-6 * want
    P["cell"][100] = 5
    P["off"][1][7] = 0.75
    ctx.deposit_mass(P, rho)
    assert ctx.status()["flag_names"] == ["offset_range"]
    P["off"][1][7] = 0.25
    P["species"][3] = 9
    ctx.deposit_mass(P, rho)
    assert ctx.status()["flag_names"] == ["bad_cell"]
    P["species"][3] = 0
    P["mom"][2][11] = float("nan")
    ctx.drag_source(P, F, w.dt, fr)
    assert ctx.status()["flag_names"] == ["nonfinite"]


def test_captured_calls_hold_no_sort_workspace():
    """A deposit captured by the caller replays correctly after larger calls
    have replaced the context's sort workspace."""
    from paper_1908_10793_amd import dust
    w = _workload("box_ragged", "f32")
    ctx = dust.context_for(w)
    P, F = dust.upload(w, ctx)
    imp = [torch.rand(w.n, device="cuda") for _ in F["dep"]]
    dep = [torch.zeros_like(d) for d in F["dep"]]
    G = dict(F, dep=dep)
    ctx.deposit(P, imp, G)           # eager: reserves the workspace
    ref = [d.clone() for d in dep]
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        for d in dep:
            d.zero_()
        ctx.deposit(P, imp, G)
    big = {k: ([t.repeat(3) for t in v] if isinstance(v, list) else v.repeat(3)) for k, v in P.items()}
    ctx.deposit(big, [q.repeat(3) for q in imp], dict(F, dep=[torch.zeros_like(d) for d in dep]))
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(dep, ref):
            assert float((a - b).abs().max()) <= 1e-5 * float(b.abs().max())
