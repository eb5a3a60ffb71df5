"""The face moments of the sweep kernel, taken over whole faces of cells inside
the domain and piece by piece elsewhere: the gradient against the general
kernel's, which takes every piece by itself.  Both sum the same integrals; the
rounding of some hundred terms stays below 1e-12 of the largest component, and
1e-10 is asked for."""
import numpy as np
import pytest

import vdgen
from gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_07175_amd as vd
    vd.load()


def _hub(seed):
    """A large cell inside the domain, and others around it."""
    d = vdgen.sphere_sites(24, seed=seed)
    rng = np.random.default_rng(seed)
    far = rng.random((300, 3))
    far = far[np.linalg.norm(far - 0.5, axis=1) > 0.45]
    return np.vstack([[[0.5, 0.49, 0.51]], 0.5 + 0.36 * d, far])


CASES = {
    "one cell": (lambda: vdgen.uniform_cube_sites(1, seed=1), lambda: vdgen.kuhn_cube_grid(2)),
    "boundary cells": (lambda: vdgen.uniform_cube_sites(12, seed=2), lambda: vdgen.kuhn_cube_grid(3)),
    "inside and boundary": (lambda: vdgen.uniform_cube_sites(900, seed=3), lambda: vdgen.kuhn_cube_grid(4)),
    "more than 64 pieces inside": (lambda: _hub(4), lambda: vdgen.kuhn_cube_grid(8)),
    "notch": (lambda: vdgen.l_block_sites(400, seed=5), lambda: vdgen.l_block(6)),
}


@pytest.mark.parametrize("density", [None, (1.0, 0.5, -0.3, 0.2, 0.4, 0.1, -0.2, 0.3, 0.05, 0.6)], ids=["", "density"])
@pytest.mark.parametrize("name", CASES)
def test_gradient_of_whole_faces(name, density):
    import torch
    import paper_2509_07175_amd as vd
    sites, dom = (f() for f in CASES[name])
    n = len(sites)
    log(f"cell moments: {name}, n={n} m={dom.m} density={density is not None}")
    s = torch.as_tensor(np.ascontiguousarray(sites), dtype=torch.float64, device="cuda")
    d = vd.Domain.from_vdgen(dom)
    g = torch.Generator().manual_seed(7)
    up = [torch.randn(n, generator=g, dtype=torch.float64).cuda(), torch.randn(n, 3, generator=g, dtype=torch.float64).cuda(),
          torch.randn(n, generator=g, dtype=torch.float64).cuda()]
    out = []
    kw = {} if density is None else {"density": density}
    for cache in (1, 0):
        grid = vd.build_grid(s, bbox=(0, 0, 0, 1, 1, 1))
        c = vd.clip_cells(grid, d, vd.Options.default(want_grad=1, site_cache=cache, **kw))
        out.append(c.backward(*up).clone())
        if name.startswith("more"):
            assert int(np.bincount(vd.pieces_as_result(c.view())["piece_site"]).max()) > 64
    torch.cuda.synchronize()
    scale = float(out[1].abs().max())
    diff = float((out[0] - out[1]).abs().max())
    log(f"max |diff| {diff:.2e} of {scale:.2e}")
    assert diff <= 1e-10 * max(scale, 1e-12)
