"""The sweep kernel of the default 3D clip at the edges of its range, against
the oracle: few sites, the LDS copy empty / full / cut to a prefix of buckets /
given up (too dense), cells with more corners or planes than lanes and plane
slots (handed to the general kernel), simplex queues beyond their LDS part, and
cells that reach out of a non-convex domain (certified piece by piece)."""
import numpy as np
import pytest

import vdgen
from gpu_util import assert_parity, log, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_07175_amd as vd
    vd.load()


def _uniform(n, seed):
    return vdgen.uniform_cube_sites(n, seed=seed, jitter=1e-7)


def _ball(n, seed, radius, at=(0.5, 0.45, 0.55)):
    """A site with n neighbours on a sphere around it: a cell of n faces."""
    d = vdgen.sphere_sites(n, seed=seed)
    return np.vstack([[at], np.asarray(at) + radius * d * (1 + 1e-3 * np.random.default_rng(seed).random((n, 1)))])


def _dense(n, seed, width):
    """n sites in a cube of that width, and 40 in the rest of the domain."""
    return np.vstack([0.4 + width * _uniform(n, seed), _uniform(40, seed + 1)])


CASES = {
    "1 site": lambda: (_uniform(1, 1), vdgen.kuhn_cube_grid(1)),
    "3 sites, long simplex queues": lambda: (_uniform(3, 2), vdgen.kuhn_cube_grid(6)),
    "64 sites": lambda: (_uniform(64, 3), vdgen.kuhn_cube_grid(2)),
    "129 sites": lambda: (_uniform(129, 4), vdgen.kuhn_cube_grid(2)),
    "513 sites": lambda: (_uniform(513, 5), vdgen.kuhn_cube_grid(3, jitter=0.1, seed=5)),
    "33 faces": lambda: (_ball(33, 6, 0.2), vdgen.kuhn_cube_grid(2)),
    "40 faces": lambda: (_ball(40, 7, 0.2), vdgen.kuhn_cube_grid(2)),
    "60 faces": lambda: (_ball(60, 8, 0.2), vdgen.kuhn_cube_grid(2)),
    "no copy": lambda: (_dense(1500, 9, 2e-3), vdgen.kuhn_cube_grid(2)),
    "prefix of a copy": lambda: (_dense(700, 10, 0.1), vdgen.kuhn_cube_grid(3)),
    "notch": lambda: (vdgen.l_block_sites(150, seed=11), vdgen.l_block(4)),
    "cavity": lambda: (_cavity_sites(12), vdgen.cube_with_cavity(6)),
}


def _cavity_sites(seed):
    s = _uniform(400, seed)
    return s[~np.all((s > 1 / 3) & (s < 2 / 3), axis=1)]


@pytest.mark.parametrize("name", CASES)
def test_sweep_against_the_oracle(oracle_mod, name):
    sites, dom = CASES[name]()
    log(f"sweep: {name}, n={len(sites)} m={dom.m}")
    ref = oracle_mod.compute(sites, dom, brute=False)
    mom = oracle_mod.site_moments(ref, sites)
    gpu = run_gpu(sites, dom)
    assert gpu["info"]["status"] == 0
    assert_parity(gpu, ref, mom, len(sites))
    # the general kernel (no LDS copy) gives the same pieces
    gen = run_gpu(sites, dom, site_cache=0)
    for k in ("piece_site", "piece_simplex"):
        assert np.array_equal(gpu["res"][k], gen["res"][k])
    assert np.array_equal(gpu["nbr_off"], gen["nbr_off"]) and np.array_equal(gpu["nbr"], gen["nbr"])
