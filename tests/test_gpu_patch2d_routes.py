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


def burst(srv, items):
    import time
    t = time.perf_counter()
    tickets = [srv.submit(p, **o) for p, o in items]
    out = [srv.wait(k, timeout=100) for k in tickets]
    t = time.perf_counter() - t
    for k in tickets:
        srv.release(k)
    return t * 1e3, out


def test_server_large_requests_join_small_ones(cf):
    """Ticks that run as one for small requests are not as long in steps when
    large ones have joined: their device time stays near the 2 ms meant."""
    import time
    prims = [Box((-BIG, -BIG, -BIG), (BIG, 1, BIG), 1)]
    small, large = vacuum(13, 14, WALLS, "TM+TE"), vacuum(180, 160, WALLS, "TM+TE", n_harm=40, prims=prims)
    large = large.replace(s_hi=(43, 43, 1))
    ps, pl = cf.Problem.from_workload(small), cf.Problem.from_workload(large)
    halos = []
    with cf.Server(16 << 30, precision="fp32") as srv:
        for _ in range(2):
            long = srv.submit(ps, **RUN, n_steps=400000, pol=small.pol)
            time.sleep(0.05)
            tickets = [srv.submit(pl, **RUN, n_steps=1500, pol=large.pol) for _ in range(6)]
            longest, last, joined = 0.0, srv.stats(), False
            while not joined or srv.poll(tickets[-1])[0] != "done":
                now = srv.stats()
                if now["clock_steps"] != last["clock_steps"]:
                    longest = max(longest, now["busy_s"] - last["busy_s"])
                    last = now
                joined = joined or srv.poll(tickets[-1])[0] == "running"
            srv.cancel(long)
            for t in tickets:
                r = srv.wait(t, timeout=100)
                assert r["fused"]
                halos.append(r["tile_halo"])
        print(f"longest tick {longest * 1e3:.1f} ms", flush=True)
        assert longest < 8e-3 and min(halos) > 8


@pytest.mark.parametrize("beside", ["3d", "tiles"])
def test_server_beside_other_requests(cf, beside):
    """Requests on patches next to a 3D one or one on tiles keep launches of many
    steps: results as alone, in no more time than with everything on tiles."""
    from casimir_inputs.configs import sphere_plate3d
    prims = [Box((-BIG, -BIG, -BIG), (BIG, 1, BIG), 1)]
    wls = [vacuum(61, 37, WALLS, "TM+TE"), vacuum(150, 120, WALLS, "TM+TE", n_harm=4, prims=prims).replace(s_hi=(43, 43, 1)),
           vacuum(260, 200, WALLS, "TM+TE", n_harm=4, prims=prims).replace(s_hi=(43, 43, 1))]
    items = [(cf.Problem.from_workload(w), dict(RUN, n_steps=n, pol=w.pol)) for w, n in zip(wls, (700, 900, 801))]
    refs = [p.solve(split=True, precision="fp32", **o) for p, o in items]
    if beside == "3d":
        w = sphere_plate3d(64, 1.0, n_harm=2)
        other = (cf.Problem.from_workload(w), dict(sigma=w.sigma, courant=w.courant, n_steps=200000, pol="3D", kernel=w.kernel))
    else:
        w = vacuum(180, 160, WALLS, "TM+TE")
        ids = {k: v.copy() for k, v in w.comp_ids.items()}
        for v in ids.values():
            v.reshape(160, 180)[100:120, 100:150] = 2
            v.reshape(160, 180)[130:150, 100:150] = 3
        w = w.replace(eps=[1.0, PEC, 3.1, 2.0], mu=[1.0, 1.0, 1.7, 1.3], comp_ids=ids)
        other = (cf.Problem.from_workload(w), dict(RUN, n_steps=300000, pol=w.pol))
    ms = {}
    for variant in (0, 13):
        with cf.Server(16 << 30, precision="fp32", tile_variant=variant) as srv:
            t = srv.submit(other[0], **other[1])
            times = [burst(srv, items) for _ in range(5)]
            ms[variant] = min(x[0] for x in times)
            patched = times[0][1] if variant == 0 else patched
            srv.cancel(t)
            for _, out in times:
                for r, ref in zip(out, refs):
                    assert r["fused"] and np.array_equal(r["per_channel"], ref["per_channel"])
                    assert variant == 0 or r["tile_halo"] == 8
    print(beside, ms, flush=True)
    assert ms[0] <= 1.1 * ms[13] and all(r["tile_halo"] > 8 for r in patched)


def test_batch_of_few_channels(cf):
    """Groups of unlike shapes and rims that leave compute units idle run beside
    each other: a batch takes no longer than its tiles, and gives each problem
    what its own split solve gives."""
    prims = [Box((-BIG, -BIG, -BIG), (BIG, 1, BIG), 1)]
    wls = [vacuum(260, 200, WALLS, "TM+TE", n_harm=2, prims=prims).replace(s_hi=(43, 43, 1)), vacuum(61, 37, WALLS, "TM+TE", n_harm=2),
           vacuum(300, 300, WALLS, "TM+TE", n_harm=2, prims=prims).replace(s_hi=(43, 43, 1))]
    probs = [cf.Problem.from_workload(w) for w in wls]
    o = dict(RUN, n_steps=600, pol="TM+TE", precision="fp32")
    refs = [p.solve(split=True, **o) for p in probs]
    ms = {}
    for variant in (0, 7, 13):
        for graph in (False, True):
            for _ in range(4):
                rs = cf.batch_solve(probs, graph=graph, tile_variant=variant, **o)
                for r, ref in zip(rs, refs):
                    assert np.array_equal(r["per_channel"], ref["per_channel"]) and tiled(r, "fp32") == (variant > 0)
                ms[variant, graph] = min(ms.get((variant, graph), 1e9), rs[0]["device_ms"])
    print(ms, flush=True)
    assert ms[0, True] <= 1.15 * min(ms[v, True] for v in (7, 13))
