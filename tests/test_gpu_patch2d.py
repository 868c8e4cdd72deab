"""The patch kernel of the Cartesian 2D problems against the split half-step
kernels, bit for bit: every shape the plan can take (lists of one patch to the
largest), partial last patches, periodic edges, conductors that leave holes in
the patch list, one and several materials of either kind, both polarizations
and precisions.  The two paths evaluate the same operations per cell, so the
tolerance is zero."""
import numpy as np
import pytest

from casimir_inputs.geometry import PEC, Box, Workload, rasterize

pytestmark = pytest.mark.gpu

BIG = 1e30


@pytest.fixture(scope="module")
def cf():
    import torch
    assert torch.cuda.is_available()
    import paper_0906_5170_amd as cf
    cf.load()
    return cf


def problem(nx, ny, bc, media="vacuum", slab=1, pol="TM+TE", n_steps=130):
    """A stress surface between conductors: a strip of `slab` rows, a block in
    a corner and a pillar (holes in the patch list); `media` adds dielectric or
    magnetic parts.  Enough steps for the near walls to answer."""
    prims = [Box((-BIG, -BIG, -BIG), (BIG, slab, BIG), 1), Box((nx - 4, ny - 4, -BIG), (BIG, BIG, BIG), 1),
             Box((5, slab + 4, -BIG), (7, slab + 6, BIG), 1)]
    eps, mu = [1.0, PEC], [1.0, 1.0]
    if media == "filled":                    # one dielectric everywhere
        eps = [2.3, PEC]
    if media == "mixed":                     # two dielectrics, one of them magnetic
        prims.append(Box((nx - 3, slab + 2, -BIG), (nx - 1, ny - 5, BIG), 2))
        eps, mu = [1.0, PEC, 3.1], [1.0, 1.0, 1.7]
    if media == "mu5":                       # one dielectric, two permeabilities
        prims.append(Box((nx - 3, slab + 2, -BIG), (nx - 1, ny - 5, BIG), 2))
        eps, mu = [1.0, PEC, 1.0], [1.0, 1.0, 5.0]
    if media == "three":                     # three permeabilities
        prims += [Box((nx - 3, slab + 2, -BIG), (nx - 1, ny - 5, BIG), 2), Box((0, ny - 4, -BIG), (4, ny - 2, BIG), 3)]
        eps, mu = [1.0, PEC, 1.0, 1.0], [1.0, 1.0, 5.0, 2.0]
    if media == "pmc":                       # a magnetic conductor (H held at 0)
        prims.append(Box((nx - 3, slab + 2, -BIG), (nx - 1, ny - 5, BIG), 2))
        eps, mu = [1.0, PEC, 1.0], [1.0, 1.0, PEC]
    return Workload(name="patch2d", ndim=2, shape=(nx, ny, 1), res=8.0, bc=bc, pml_cells=(0, 0, 0), eps=eps, mu=mu,
                    comp_ids=rasterize((nx, ny, 1), prims), s_lo=(3, slab + 2, 0), s_hi=(9, slab + 8, 1), n_harm=3,
                    force_axis=0, sigma=0.9, courant=0.5, n_steps=n_steps, pol=pol, kernel="general")


def solve(p, wl, precision, **kw):
    return p.solve(sigma=wl.sigma, courant=wl.courant, n_steps=wl.n_steps, pol=wl.pol, kernel=wl.kernel,
                   precision=precision, keep_gamma=True, **kw)


def both(cf, wl, precision, patch=True, **kw):
    p = cf.Problem.from_workload(wl)
    a, b = solve(p, wl, precision, **kw), solve(p, wl, precision, split=True)
    assert a["fused"] and not b["fused"]
    # a patch launch takes more steps than a tile launch (8 in FP32, 4 in FP64)
    assert patch is None or (a["tile_halo"] > (8 if precision == "fp32" else 4)) == patch, a["tile_halo"]
    for key in ("per_channel", "gamma"):
        assert np.all(np.isfinite(a[key])) and np.any(a[key] != 0.0), key
        assert np.array_equal(a[key], b[key]), (wl.shape, wl.bc, precision, key)
    assert a["force"] == b["force"]
    return p, a


W = ("pec", "pec", "periodic")
P = ("periodic", "periodic", "periodic")
SHAPES = [((13, 14), W), ((16, 16), P), ((23, 19), ("pec", "pec", "periodic")), ((24, 31), ("periodic", "pec", "periodic")),
          ((31, 24), ("pec", "periodic", "periodic")), ((61, 37), W), ((97, 83), W), ((120, 100), ("periodic", "pec", "periodic"))]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("media", ["vacuum", "filled", "mixed", "pmc", "mu5", "three"])
@pytest.mark.parametrize("shape,bc", SHAPES)
def test_bitwise(cf, shape, bc, media, precision):
    # 8000 cells and more fit no shape in FP64 or with several materials
    both(cf, problem(*shape, bc, media), precision, patch=True if shape[0] < 80 else None)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("pol", ["TM", "TE"])
@pytest.mark.parametrize("media", ["vacuum", "mixed"])
def test_small_one_polarization(cf, media, pol, precision):
    """Small grids start their channels in the patch kernel; one polarization
    alone, and enough channels that both do not share a launch."""
    both(cf, problem(29, 23, W, media, pol=pol), precision)
    both(cf, problem(29, 23, W, media).replace(n_harm=20), precision)


@pytest.mark.parametrize("pol", ["TM", "TE"])
@pytest.mark.parametrize("shape,slab,media", [((150, 120), 1, "vacuum"), ((180, 160), 1, "vacuum"),
                                              ((176, 170), 1, "filled"), ((400, 200), 150, "vacuum"),
                                              ((110, 100), 1, "mixed"), ((170, 160), 1, "mu5"), ((150, 120), 1, "pmc")])
def test_largest_shapes(cf, shape, slab, media, pol):
    """Grids that take the largest FP32 shapes, and one mostly of conductor."""
    both(cf, problem(*shape, W, media, slab, pol, n_steps=60), "fp32")


@pytest.mark.parametrize("shape,bc,slab,pol", [
    ((260, 200), W, 1, "TM+TE"), ((200, 260), W, 1, "TM"), ((512, 96), ("periodic", "pec", "periodic"), 1, "TM+TE"),
    ((96, 512), ("pec", "periodic", "periodic"), 1, "TE"), ((400, 300), W, 150, "TM+TE"), ((417, 203), W, 2, "TE")])
@pytest.mark.parametrize("media", ["vacuum", "mu5", "pmc"])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_parts(cf, shape, bc, slab, pol, precision, media):
    """Grids beyond one compute unit go in parts, cut along either axis, over
    periodic edges too; several launches, the last one shorter."""
    # FP64 lists of a grid without conductor may find no room: tiles
    both(cf, problem(*shape, bc, media, slab, pol, n_steps=75), precision,
         patch=True if media == "vacuum" and (precision == "fp32" or slab > 100) else None)


def test_parts_waves_graph_and_stop(cf):
    wl = problem(260, 200, W, n_steps=150)
    p, a = both(cf, wl, "fp32")
    for kw in (dict(graph=True), dict(max_resident=5), dict(graph=True, max_resident=7), dict(time_stencil=True)):
        for _ in range(2):
            r = solve(p, wl, "fp32", **kw)
            assert np.array_equal(r["per_channel"], a["per_channel"]) and np.array_equal(r["gamma"], a["gamma"]), kw
    s = p.solve(sigma=wl.sigma, courant=wl.courant, n_steps=wl.n_steps, pol=wl.pol, kernel=wl.kernel,
                precision="fp32", stop_tol=1e6, stop_every=40)
    assert 40 < s["n_steps_run"] < wl.n_steps
    t = solve(p, wl.replace(n_steps=s["n_steps_run"]), "fp32")
    assert np.array_equal(t["per_channel"], s["per_channel"])


def test_beyond_the_shapes(cf):
    """A grid no shape covers (several materials) stays with the tiles."""
    both(cf, problem(180, 160, W, "mixed", n_steps=30), "fp32", patch=False)


def test_waves_graph_and_stop(cf):
    """Channel waves, graph capture (replayed with eager work between) and the
    convergence stop leave the results what they are."""
    wl = problem(61, 37, W, n_steps=400)
    p, a = both(cf, wl, "fp32")
    for kw in (dict(graph=True), dict(max_resident=5), dict(graph=True, max_resident=5), dict(time_stencil=True)):
        for _ in range(2):
            r = solve(p, wl, "fp32", **kw)
            assert np.array_equal(r["per_channel"], a["per_channel"]) and np.array_equal(r["gamma"], a["gamma"]), kw
    s = p.solve(sigma=wl.sigma, courant=wl.courant, n_steps=wl.n_steps, pol=wl.pol, kernel=wl.kernel,
                precision="fp32", stop_tol=1e6, stop_every=50)
    assert 50 < s["n_steps_run"] < wl.n_steps
    t = solve(p, wl.replace(n_steps=s["n_steps_run"]), "fp32")
    assert np.array_equal(t["per_channel"], s["per_channel"])


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("graph", [False, True])
def test_batch(cf, graph, precision):
    """A batch of problems of both kinds (patches of several shapes, tiles)
    gives every problem what its own split solve gives, twice."""
    wls = [problem(13, 14, W), problem(97, 83, W, "filled"), problem(260, 200, W), problem(61, 37, W, "mixed"),
           problem(24, 31, ("periodic", "pec", "periodic")), problem(180, 160, W, "mixed")]
    wls = [w.replace(n_steps=70) for w in wls]
    probs = [cf.Problem.from_workload(w) for w in wls]
    o = dict(sigma=0.9, courant=0.5, n_steps=70, pol="TM+TE", kernel="general", precision=precision)
    for some in (probs, probs[:2], probs[2:3], probs[5:], probs):
        for r, p in zip(cf.batch_solve(some, graph=graph, **o), some):
            b = p.solve(split=True, **o)
            assert r["fused"] and np.array_equal(r["per_channel"], b["per_channel"])


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_server(cf, precision):
    """Requests on patches and on tiles, joining one after another, get what
    their own split solves give; so does one that stops early."""
    wls = [problem(13, 14, W), problem(97, 83, W, "filled"), problem(61, 37, W, "mixed"), problem(260, 200, W),
           problem(61, 37, W), problem(24, 31, ("periodic", "pec", "periodic")), problem(180, 160, W, "mixed")]
    steps = [400, 61, 250, 90, 300, 77, 83]
    probs = [cf.Problem.from_workload(w) for w in wls]
    o = [dict(sigma=0.9, courant=0.5, n_steps=n, pol="TM+TE", kernel="general", precision=precision) for n in steps]
    o[4].update(stop_tol=1e6, stop_every=40)
    srv = cf.Server(2 << 30, precision=precision)
    for some in (range(3), range(2, 4), range(7)):
        tickets = [srv.submit(probs[k], **o[k]) for k in some]
        for k, t in zip(some, tickets):
            r = srv.wait(t, timeout=100)
            ref = dict(sigma=0.9, courant=0.5, pol="TM+TE", kernel="general", precision=precision)
            b = probs[k].solve(split=True, n_steps=r["n_steps_run"], **ref)
            assert r["n_steps_run"] == steps[k] if k != 4 else 40 < r["n_steps_run"] < 300
            assert r["fused"] and np.array_equal(r["per_channel"], b["per_channel"]), k
            srv.release(t)
    srv.close()


def test_batch_of_parts(cf):
    """Problems whose rims differ do not share launches;
    enough steps for waves to cross the cuts and return."""
    wls = [problem(400, 300, W, slab=150, n_steps=500), problem(260, 200, W, n_steps=500)]
    probs = [cf.Problem.from_workload(w) for w in wls]
    o = dict(sigma=0.9, courant=0.5, n_steps=500, pol="TM+TE", kernel="general", precision="fp32")
    halos = {p.solve(**o)["tile_halo"] for p in probs}
    assert len(halos) == 2, halos
    for some in (probs, probs[::-1]):
        for r, p in zip(cf.batch_solve(some, **o), some):
            assert np.array_equal(r["per_channel"], p.solve(split=True, **o)["per_channel"])


def test_parts_long(cf):
    """Waves that cross the cuts many times."""
    for shape, slab, media in (((260, 200), 1, "vacuum"), ((400, 300), 150, "vacuum"), ((260, 200), 1, "mu5")):
        both(cf, problem(*shape, W, media, slab, n_steps=1500).replace(n_harm=1), "fp32")
