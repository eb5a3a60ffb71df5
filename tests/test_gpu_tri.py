"""The sweep kernel of the default surface clip at the edges of its range,
against the oracle and the searched kernel: few sites, triangles smaller and
larger than the cells, more sites around a triangle than its LDS copy holds, a
piece of more than 16 vertices met after others of its triangle were written
(they are voided and the triangle is redone), sites off the surface."""
import numpy as np
import pytest

import vdgen
from gpu_util import assert_csr, assert_parity, log, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_07175_amd as vd
    vd.load()


def _area(dom):
    q = dom.verts[dom.simplices]
    return float(0.5 * np.linalg.norm(np.cross(q[:, 1] - q[:, 0], q[:, 2] - q[:, 0]), axis=1).sum())


def _hub(seed, m=20, at=(0.3, 0.12), r=0.08):
    """A site with m others on a circle around it, in the plane of the L, and
    60 uniform ones elsewhere: its cell is one polygon of m sides, away from
    its triangle's centroid and corners."""
    rng = np.random.default_rng(seed)
    t = 2 * np.pi * (np.arange(m) + 0.2 * rng.random(m)) / m
    ring = np.stack([at[0] + r * np.cos(t), at[1] + r * np.sin(t)], 1) * (1 + 1e-4 * rng.random((m, 1)))
    far = rng.random((60, 2))
    far = far[np.hypot(far[:, 0] - at[0], far[:, 1] - at[1]) > 2.2 * r]
    p = np.vstack([[at], ring, far])
    return np.hstack([p, 1e-6 * rng.random((len(p), 1))])


def _clump(seed):
    """600 sites in a patch of the sphere that holds 1/1000 of it, 40 elsewhere."""
    s = vdgen.sphere_sites(640, seed=seed)
    t = np.array([0.3, -0.5, 0.8]) + 0.05 * s[:600]
    return np.vstack([t / np.linalg.norm(t, axis=1, keepdims=True), s[600:]])


CASES = {
    "1 site": lambda: (vdgen.planar_l_sites(1, seed=1), vdgen.planar_l_polygon(4)),
    "2 sites": lambda: (vdgen.sphere_sites(2, seed=2), vdgen.icosphere(2)),
    "17 sites, fine mesh": lambda: (vdgen.sphere_sites(17, seed=3), vdgen.icosphere(4)),
    "coarse mesh": lambda: (vdgen.sphere_sites(400, seed=4), vdgen.icosphere(1)),
    "129 sites, 20 triangles": lambda: (vdgen.sphere_sites(129, seed=5), vdgen.icosphere(0)),
    "clump": lambda: (_clump(6), vdgen.icosphere(3)),
    "polygon of 20 sides": lambda: (_hub(7), vdgen.planar_l_polygon(2)),
    "polygon of 15 sides": lambda: (_hub(8, m=15), vdgen.planar_l_polygon(2)),
    "off the surface": lambda: (0.5 * vdgen.sphere_sites(300, seed=9) * np.linspace(0.1, 1.9, 300)[:, None],
                                vdgen.icosphere(3)),
}


@pytest.mark.parametrize("name", CASES)
def test_tri_against_the_oracle(oracle_mod, name):
    sites, dom = CASES[name]()
    area = _area(dom)
    log(f"surface sweep: {name}, n={len(sites)} m={dom.m}")
    box = (-1.01, -1.01, -1.01, 1.01, 1.01, 1.01)
    ref = oracle_mod.compute(sites, dom, brute=False)
    mom = oracle_mod.site_moments(ref, sites)
    gpu = run_gpu(sites, dom, bbox=box, surface_area=area)
    assert gpu["info"]["status"] == 0
    assert_parity(gpu, ref, mom, len(sites))
    assert_csr(gpu, len(sites))
    assert abs(gpu["mass"].sum() - area) <= 1e-12 * area
    # the searched kernel (no LDS copy) gives the same pieces
    gen = run_gpu(sites, dom, bbox=box, surface_area=area, site_cache=0)
    for k in ("piece_site", "piece_simplex"):
        assert np.array_equal(gpu["res"][k], gen["res"][k])
    assert np.array_equal(gpu["nbr_off"], gen["nbr_off"]) and np.array_equal(gpu["nbr"], gen["nbr"])
