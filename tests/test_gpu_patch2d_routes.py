"""Which calls the 2D patch kernel takes and what it reports of them: channel
waves of one polarization, batches of many small problems, grids in parts by
their number of channels, served requests beside others."""
import numpy as np
import pytest

from casimir_inputs.geometry import PEC, Box, Workload, rasterize

pytestmark = pytest.mark.gpu

BIG = 1e30
RUN = dict(sigma=0.9, courant=0.5, kernel="general")


@pytest.fixture(scope="module")
def cf():
    import torch
    assert torch.cuda.is_available()
    import paper_0906_5170_amd as cf
    cf.load()
    return cf


def vacuum(nx, ny, bc, pol, s_hi=None, n_harm=3, prims=()):
    return Workload(name="route", ndim=2, shape=(nx, ny, 1), res=8.0, bc=bc, pml_cells=(0, 0, 0), eps=[1.0, PEC],
                    mu=[1.0, 1.0], comp_ids=rasterize((nx, ny, 1), list(prims)), s_lo=(3, 0 if s_hi else 3, 0),
                    s_hi=s_hi or (9, 9, 1), n_harm=n_harm, force_axis=0, sigma=0.9, courant=0.5, n_steps=60, pol=pol,
                    kernel="general")


def tiled(r, precision):
    """Whether the tiles advanced a 2D result (8 steps a launch at most, 4 in FP64)."""
    return r["fused"] and r["tile_halo"] <= (8 if precision == "fp32" else 4)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_waves_of_one_polarization(cf, precision):
    """Without a conductor every cell is in a patch: the cells advanced are all
    cells, whatever polarizations a wave of channels holds."""
    wl = vacuum(24, 36, ("periodic", "periodic", "periodic"), "TM+TE")
    p = cf.Problem.from_workload(wl)
    o = dict(RUN, n_steps=60, pol=wl.pol, precision=precision)
    for kw in ({}, dict(max_resident=5), dict(max_resident=3)):
        r = p.solve(**o, **kw)
        assert not tiled(r, precision) and r["advanced_cell_updates"] == r["cell_updates"], kw


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [8, 72])
def test_batch_of_strips(cf, n, precision):
    """Strips of six channels each: the patch kernel's heads and items of many
    of them need more room than their tiles' work items have."""
    wl = vacuum(20, 8, ("pec", "periodic", "periodic"), "TE", s_hi=(9, 8, 1), n_harm=1)
    p = cf.Problem.from_workload(wl)
    o = dict(RUN, n_steps=60, pol="TE", precision=precision)
    ref = p.solve(split=True, **o)
    for r in cf.batch_solve([p] * n, **o):
        assert r["n_channels"] == 6 and tiled(r, precision) == (n > 40)
        assert np.array_equal(r["per_channel"], ref["per_channel"])


def best_ms(p, o, **kw):
    return min(p.solve(**o, **kw)["device_ms"] for _ in range(4))


def check_speed(cf, wl, slack, n_steps=200):
    """The route left to the library is not slower than the tiles' best shape."""
    p = cf.Problem.from_workload(wl)
    o = dict(RUN, n_steps=n_steps, pol=wl.pol, precision="fp32")
    tiles = []
    for v in range(1, 20):
        r = p.solve(**o, tile_variant=v)
        if r["tile_variant"] == v:
            tiles.append(best_ms(p, o, tile_variant=v))
    mine = best_ms(p, o)
    print(wl.shape, wl.n_harm, f"{mine:.3f} ms, tiles {min(tiles):.3f}", flush=True)
    assert len(tiles) > 2 and mine <= slack * min(tiles), (mine, tiles)


WALLS = ("pec", "pec", "periodic")


@pytest.mark.parametrize("shape", [(300, 300), (440, 330)])
def test_speed_of_parts(cf, shape):
    """Large grids in parts, more channels than the device takes at once."""
    prims = [Box((-BIG, -BIG, -BIG), (BIG, 1, BIG), 1)]
    check_speed(cf, vacuum(*shape, WALLS, "TM+TE", n_harm=20, prims=prims).replace(s_hi=(43, 43, 1)), 1.1)


@pytest.mark.parametrize("n_harm,slack", [(1, 1.3), (2, 1.15), (4, 1.1)])
@pytest.mark.parametrize("shape", [(260, 200), (300, 300)])
def test_speed_of_parts_with_few_channels(cf, shape, n_harm, slack):
    """16 channels a harmonic leave most compute units idle: the parts chosen
    are those with the shortest step, not the least work.  (One harmonic: a
    step of the smallest parts that fit is as long as the tiles' launches.)"""
    prims = [Box((-BIG, -BIG, -BIG), (BIG, 1, BIG), 1)]
    check_speed(cf, vacuum(*shape, WALLS, "TM+TE", n_harm=n_harm, prims=prims).replace(s_hi=(43, 43, 1)), slack, 600)
