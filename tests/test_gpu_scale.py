"""The clips have no length scale of their own: sites and domain times a power of
two give the same diagram, its moments times powers of that (every operation
scales exactly, short of the ends of the exponents)."""
import numpy as np
import pytest

import vdgen
from gpu_util import log, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_07175_amd as vd
    vd.load()


def _run(sites, dom, scale, lo, **kw):
    d = vdgen.Domain(verts=dom.verts * scale, simplices=dom.simplices, adj=dom.adj, dim=dom.dim)
    w = kw.pop("weights", None)
    return run_gpu(sites * scale, d, bbox=tuple(lo * scale for _ in range(3)) + (scale,) * 3,
                   weights=None if w is None else w * scale ** 2, **kw)


@pytest.mark.parametrize("power", [-85, -60, 60])
@pytest.mark.parametrize("what", ["solid", "weights", "surface"])
def test_scaled(what, power):
    scale = 2.0 ** power
    if what == "surface":
        sites, dom, lo, kw = vdgen.sphere_sites(300, seed=4), vdgen.icosphere(2), -1.0, {}
    else:
        sites, dom, lo, kw = vdgen.uniform_cube_sites(700, seed=5, jitter=1e-7), vdgen.kuhn_cube_grid(2), 0.0, {}
        if what == "weights":
            kw["weights"] = 1e-3 * np.random.default_rng(6).random(len(sites))
    ref, got = (_run(sites, dom, f, lo, **kw) for f in (1.0, scale))
    assert got["info"]["status"] == 0
    err = np.abs(got["mass"] / scale ** (2 if what == "surface" else 3) - ref["mass"]) / ref["mass"].max()
    log(f"{what} 2^{power}: {err.max():.1e}")
    assert err.max() < 1e-12
    assert np.array_equal(got["nbr_off"], ref["nbr_off"]) and np.array_equal(got["nbr"], ref["nbr"])
