"""The patch kernel of the reduced problems (cylindrical, k_z, Bloch) against
the split half-step kernels, bit for bit: grids that leave every shape a
partial last patch, grids one patch wide, the largest a shape covers, walls
and periodic edges, several materials, and both precisions.  The two paths
evaluate the same operations per cell, so the tolerance is zero."""
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


def block_problem(nx, ny, bc, kx=(), n_steps=150):
    """Two dielectric blocks and a PEC strip around a stress surface; enough
    steps for every wall to answer."""
    prims = [Box((-BIG, -BIG, -BIG), (BIG, 1, BIG), 1), Box((nx - 3, 3, -BIG), (nx - 2, ny - 3, BIG), 3),
             Box((5, 5, -BIG), (7, 7, BIG), 2)]
    kz = (0.7, 2.9)
    return Workload(name="patch", ndim=2, shape=(nx, ny, 1), res=8.0, bc=bc, pml_cells=(0, 0, 0),
                    eps=[1.0, PEC, 3.3, 2.2], mu=[1.0, 1.0, 1.0, 1.4], comp_ids=rasterize((nx, ny, 1), prims),
                    s_lo=(3, 3, 0), s_hi=(9, 9, 1), n_harm=3, force_axis=0, sigma=0.9, courant=0.5,
                    n_steps=n_steps, pol="3D", kernel="general", coord="kz", kz=kz, kz_weight=(0.4, 0.3), kx=tuple(kx))


def both(cf, wl, precision):
    p = cf.Problem.from_workload(wl)
    o = dict(sigma=wl.sigma, courant=wl.courant, n_steps=wl.n_steps, pol="3D", kernel="general",
             precision=precision, keep_gamma=True)
    a, b = p.solve(**o), p.solve(split=True, **o)
    assert a["fused"] == (not wl.lorentz and "pml" not in wl.bc) and not b["fused"]
    for key in ("per_channel", "gamma"):
        assert np.all(np.isfinite(a[key])) and np.any(a[key] != 0.0), key
        assert np.array_equal(a[key], b[key]), (wl.shape, wl.bc, precision, key)
    assert a["force"] == b["force"]


WALLS = ("pec", "pec", "periodic")
KZ = [((13, 13), WALLS), ((16, 15), ("periodic", "periodic", "periodic")), ((24, 21), ("periodic", "pec", "periodic")),
      ((41, 25), ("pec", "periodic", "periodic")), ((67, 43), WALLS), ((81, 61), WALLS), ((120, 40), WALLS),
      ((100, 77), WALLS), ((13, 511), WALLS)]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shape,bc", KZ)
def test_kz(cf, shape, bc, precision):
    both(cf, block_problem(*shape, bc), precision)


@pytest.mark.parametrize("shape", [(130, 90), (160, 80)])
def test_kz_beyond_the_exchange_array(cf, shape):
    """Grids of more than 10240 cells, FP32."""
    both(cf, block_problem(*shape, WALLS), "fp32")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shape,bc_y", [((14, 13), "pec"), ((24, 22), "periodic"), ((36, 40), "pec"),
                                        ((48, 61), "pec")])
def test_bloch(cf, shape, bc_y, precision):
    both(cf, block_problem(*shape, ("periodic", bc_y, "periodic"), kx=(0.3, 0.9)), precision)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("res,length", [(10, 5.0), (16, 7.0), (23, 6.1), (31, 8.3)])
def test_cylindrical(cf, res, length, precision):
    from casimir_inputs import cyl_piston
    wl = cyl_piston(res, h_u=0.9, length_u=length, n_harm=2, m_max=3, n_steps=150)
    both(cf, wl, precision)


POLES = ((3.0, 3.0), (1.5, 5.0))


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("res,pml,poles", [(10, 0.4, POLES[:1]), (16, 0.5, ()), (21, 0.3, POLES), (28, 0.5, POLES[:1])])
def test_open_guides(cf, res, pml, poles, precision):
    """CPML on four sides (layers that end inside a patch) and up to two
    Lorentz terms; the largest grid takes E_z into LDS in FP32."""
    from casimir_inputs import kz_workload, waveguides_open_2d
    wl = waveguides_open_2d(res, 0.5, 0.25, 0.5, 0.5, pml, 1.5, poles, n_harm=3, n_steps=150)
    both(cf, kz_workload(wl, [0.7, 2.9], [0.4, 0.3]), precision)


def test_open_guides_at_the_largest_grid(cf):
    """130 x 90 cells, FP32: the CPML values and polarizations nearly fill the
    block's LDS; 64 channels need several launches at two resident channels."""
    from casimir_inputs import kz_workload, waveguides_open_2d
    wl = waveguides_open_2d(40, 0.5, 0.25, 0.25, 0.5, 0.5, 1.5, POLES[:1], n_harm=4, n_steps=150)
    wl = kz_workload(wl, [0.7, 2.9], [0.4, 0.3])
    both(cf, wl, "fp32")
    p = cf.Problem.from_workload(wl)
    o = dict(sigma=wl.sigma, courant=wl.courant, n_steps=wl.n_steps, pol="3D", kernel="general", precision="fp32")
    assert np.array_equal(p.solve(**o)["per_channel"], p.solve(max_resident=2, **o)["per_channel"])


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_open_along_one_axis(cf, precision):
    from casimir_inputs import kz_workload, slabs_open_1d
    wl = slabs_open_1d(20, 0.5, 0.25, 0.35, 0.5, 1.5, POLES, n_steps=150)
    both(cf, kz_workload(wl, [0.7, 2.9], [0.4, 0.3]), precision)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_dispersive_without_layers(cf, precision):
    wl = block_problem(37, 29, WALLS)
    both(cf, wl.replace(lorentz={2: POLES}), precision)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("kx", [(), (0.3, 0.9)])
@pytest.mark.parametrize("shape,bc,rows", [((48, 60), ("periodic", "pec", "periodic"), 31),
                                           ((72, 48), ("periodic", "periodic", "periodic"), 17),
                                           ((80, 40), WALLS, 20), ((150, 77), WALLS, 50)])
def test_conductor_holes(cf, shape, bc, rows, kx, precision):
    """A slab of conductor and one in a corner: patches without a cell that can
    change are left out of the list, across periodic edges too."""
    if kx and bc[0] != "periodic":
        pytest.skip("Bloch runs need a periodic x axis")
    nx, ny = shape
    wl = block_problem(nx, ny, bc, kx=kx, n_steps=220)
    prims = [Box((-BIG, 14, -BIG), (BIG, 14 + min(rows, ny - 22), BIG), 1), Box((nx - 13, ny - 6, -BIG), (BIG, BIG, BIG), 1),
             Box((5, 5, -BIG), (7, 7, BIG), 2)]
    both(cf, wl.replace(comp_ids=rasterize((nx, ny, 1), prims)), precision)
