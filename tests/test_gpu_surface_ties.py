"""Surface sites that repeat: the first of those at a point has the cell, the
others are empty, in every triangle alike (solids refuse such sites)."""
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


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("copies", [1, 20])
def test_repeated_sites(oracle_mod, copies, weighted):
    n = 400
    sites = vdgen.sphere_sites(n, seed=21)
    w = 1e-3 * np.random.default_rng(3).random(n) if weighted else None
    again = np.random.default_rng(2).permutation(n)[:60 if copies == 1 else 7]
    rep = np.concatenate([np.arange(n)] + [again] * copies)
    dom = vdgen.icosphere(3)
    ref = oracle_mod.compute(sites, dom, brute=False, weights=w)
    mom = oracle_mod.site_moments(ref, sites)
    gpu = run_gpu(sites[rep], dom, bbox=(-1.0,) * 3 + (1.0,) * 3, weights=None if w is None else w[rep])
    assert gpu["info"]["status"] == 0
    err = np.abs(gpu["mass"][:n] - mom["mass"])
    log(f"copies {copies} weighted {weighted}: {err.max():.1e}, mass of repeated ones {gpu['mass'][n:].max():.1e}")
    assert np.all(gpu["mass"][n:] == 0.0)
    assert np.all(err <= 1e-9 * mom["mass"].max())
    for i in range(n):
        assert list(gpu["nbr"][gpu["nbr_off"][i]:gpu["nbr_off"][i + 1]]) == list(mom["neighbors"][i])
