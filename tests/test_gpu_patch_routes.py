"""Which calls of the reduced problems the patch kernel takes: runs with the
convergence stop, whose checks cut them into spans."""
import numpy as np
import pytest

from casimir_inputs.configs import cyl_piston, stop_cyl, stop_kz

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
