"""Which calls of the reduced problems the patch kernel takes (its launches
report their steps, the other kernels 0): the grids held bit for bit against the
split kernels elsewhere, and runs with the convergence stop, whose checks cut
them into spans."""
import numpy as np
import pytest

from casimir_inputs import kz_workload, slabs_open_1d, waveguides_open_2d
from casimir_inputs.configs import cyl_piston, stop_cyl, stop_kz
from casimir_inputs.geometry import PEC, Box, Workload, rasterize

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cf():
    import torch
    assert torch.cuda.is_available()
    import paper_0906_5170_amd as cf
    cf.load()
    return cf


def best_ms(p, **o):
    import time
    out = []
    for _ in range(5):
        t = time.perf_counter()
        r = p.solve(**o)
        out.append((time.perf_counter() - t) * 1e3)
    return min(out), r


@pytest.mark.parametrize("every", [1, 4, 7, 8, 20])
@pytest.mark.parametrize("make", [stop_cyl, stop_kz, cyl_piston])
def test_spans_are_not_slower(cf, make, every):
    """Spans of any length give the uncut run's channels, in no more time than
    the global-memory kernel, which neither plans nor fills registers, takes."""
    wl = make(n_steps=240)
    p = cf.Problem.from_workload(wl)
    o = dict(sigma=wl.sigma, courant=wl.courant, n_steps=240, pol=wl.pol, kernel=wl.kernel, precision="fp64")
    ref = p.solve(**o)
    stop = dict(stop_tol=1e-300, stop_every=every)
    best, r = best_ms(p, **o, **stop)
    plain, _ = best_ms(p, **o, **stop, tile_variant=2)
    print(wl.name, every, f"{best:.2f} ms, global-memory kernel {plain:.2f}", flush=True)
    assert np.array_equal(r["per_channel"], ref["per_channel"]) and r["n_steps_run"] == 240
    assert best <= 1.25 * plain


BIG = 1e30
WALLS = ("pec", "pec", "periodic")
POLES = ((3.0, 3.0), (1.5, 5.0))


def blocks(nx, ny, bc, kx=(), conductor=0, lorentz=None):
    """Dielectric and magnetic blocks around a stress surface, a strip of PEC
    and, with `conductor`, a slab of that many rows and a corner of it."""
    prims = [Box((-BIG, -BIG, -BIG), (BIG, 1, BIG), 1), Box((5, 5, -BIG), (7, 7, BIG), 2)]
    if conductor:
        prims += [Box((-BIG, 14, -BIG), (BIG, 14 + conductor, BIG), 1), Box((nx - 13, ny - 6, -BIG), (BIG, BIG, BIG), 1)]
    else:
        prims.append(Box((nx - 3, 3, -BIG), (nx - 2, ny - 3, BIG), 3))
    return Workload(name="route", ndim=2, shape=(nx, ny, 1), res=8.0, bc=bc, pml_cells=(0, 0, 0),
                    eps=[1.0, PEC, 3.3, 2.2], mu=[1.0, 1.0, 1.0, 1.4], comp_ids=rasterize((nx, ny, 1), prims),
                    s_lo=(3, 3, 0), s_hi=(9, 9, 1), n_harm=2, force_axis=0, sigma=0.9, courant=0.5, n_steps=60, pol="3D",
                    kernel="general", coord="kz", kz=(0.7, 2.9), kz_weight=(0.4, 0.3), kx=tuple(kx), lorentz=lorentz)


def guides(res, gap, pml, poles):
    wl = waveguides_open_2d(res, 0.5, 0.25, gap, 0.5, pml, 1.5, poles, n_harm=2, n_steps=60)
    return kz_workload(wl, [0.7, 2.9], [0.4, 0.3])


def slabs(ny):
    return kz_workload(slabs_open_1d(20, 0.5, 0.25, 0.35, 0.5, 1.5, POLES, ny=ny, n_steps=60), [0.7, 2.9], [0.4, 0.3])


PER_X, PER_Y, PER = ("periodic", "pec", "periodic"), ("pec", "periodic", "periodic"), ("periodic",) * 3
KX = (0.3, 0.9)
# workload, and whether a patch shape covers it in FP32 and in FP64: a periodic
# axis is a multiple of the patch, and the patches, LDS entries, CPML values and
# polarizations fit a compute unit
ROUTES = [
    (lambda: blocks(13, 13, WALLS), True, True), (lambda: blocks(16, 15, PER), True, True),
    (lambda: blocks(24, 21, PER_X), True, True), (lambda: blocks(41, 25, PER_Y), True, False),
    (lambda: blocks(81, 61, WALLS), True, True), (lambda: blocks(100, 77, WALLS), True, True),
    (lambda: blocks(13, 511, WALLS), True, False), (lambda: blocks(160, 80, WALLS), True, False),
    (lambda: blocks(14, 13, PER_X, KX), True, True), (lambda: blocks(29, 24, PER_X, KX), False, False),
    (lambda: blocks(24, 22, PER, KX), True, True), (lambda: blocks(48, 61, PER_X, KX), True, False),
    (lambda: cyl_piston(10, h_u=0.9, length_u=5.0, n_harm=2, m_max=3, n_steps=60), True, True),
    (lambda: cyl_piston(31, h_u=0.9, length_u=8.3, n_harm=2, m_max=3, n_steps=60), True, True),
    (lambda: guides(10, 0.5, 0.4, POLES[:1]), True, True), (lambda: guides(21, 0.5, 0.3, POLES), True, True),
    (lambda: guides(28, 0.5, 0.5, POLES[:1]), True, False), (lambda: guides(40, 0.25, 0.5, POLES[:1]), True, False),
    (lambda: slabs(1), False, False), (lambda: slabs(12), True, True),
    (lambda: blocks(37, 29, WALLS, lorentz={2: POLES}), True, True),
]


def solve(p, wl, precision, **kw):
    return p.solve(sigma=wl.sigma, courant=wl.courant, n_steps=wl.n_steps, pol="3D", kernel=wl.kernel,
                   precision=precision, **kw)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("case", range(len(ROUTES)))
def test_route(cf, case, precision):
    make, fp32, fp64 = ROUTES[case]
    wl = make()
    p = cf.Problem.from_workload(wl)
    r, s = solve(p, wl, precision), solve(p, wl, precision, split=True)
    assert r["tile_halo"] == (wl.n_steps if (fp32 if precision == "fp32" else fp64) else 0) and s["tile_halo"] == 0
    assert np.any(r["per_channel"] != 0.0) and np.array_equal(r["per_channel"], s["per_channel"])
    if wl.coord == "kz" and not wl.kx:
        assert r["advanced_cell_updates"] == r["cell_updates"]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shape,bc,rows,kx", [((48, 60), PER_X, 31, ()), ((48, 60), PER_X, 31, KX), ((72, 48), PER, 17, ()),
                                              ((72, 48), PER, 17, KX), ((80, 40), WALLS, 18, ()), ((150, 77), WALLS, 50, ())])
def test_conductor_is_left_out(cf, shape, bc, rows, kx, precision):
    """The patches advanced are those around the cells outside the conductor, not
    all of the grid's."""
    wl = blocks(*shape, bc, kx=kx, conductor=rows)
    p = cf.Problem.from_workload(wl)
    r, s = solve(p, wl, precision), solve(p, wl, precision, split=True)
    live = 1 - np.mean(wl.comp_ids["Ez"] == 1)
    share = r["advanced_cell_updates"] / r["cell_updates"]
    assert r["tile_halo"] == wl.n_steps and live < share < min(0.85, live + 0.3), (live, share)
    assert np.array_equal(r["per_channel"], s["per_channel"])
