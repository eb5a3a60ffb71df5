"""Cells that the sweep kernel leaves to the searched one after it has written some
of their pieces (a cell that fits, one of whose pieces does not), and a list of
such cells in a clip that does not wait for its length, eagerly and in a graph."""
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


def _ball(n, seed, radius, at):
    """A site with n neighbours on a sphere around it: a cell of n faces."""
    d = vdgen.sphere_sites(n, seed=seed)
    return np.vstack([[at], np.asarray(at) + radius * d * (1 + 1e-3 * np.random.default_rng(seed).random((n, 1)))])


# cells of 33 faces and 62 corners, whose tips reach past a tetrahedron: a piece of
# more than 64 corners between smaller ones, in any order of the tetrahedra
CUT = [(209996, 0.08989675692734331, (0.7458430980072324, 0.6132123196139, 0.6840190478145994)),
       (366194, 0.18955949801716698, (0.6370442638350615, 0.7461799674137235, 0.3718636194345014)),
       (699930, 0.09608846457331774, (0.4091965578278303, 0.544581547600701, 0.45782116788561716)),
       (779591, 0.1787939561339319, (0.6684782286544821, 0.5652649958643663, 0.29902978747283154))]


@pytest.mark.parametrize("k", range(len(CUT)))
@pytest.mark.parametrize("grad", [0, 1])
def test_a_piece_that_does_not_fit(oracle_mod, k, grad):
    sites, dom = _ball(33, *CUT[k]), vdgen.kuhn_cube_grid(2)
    ref = oracle_mod.compute(sites, dom, brute=False)
    corners = np.diff(ref["piece_vert_off"])[ref["piece_site"] == 0]
    log(f"corners of the pieces of site 0: {corners}")
    assert corners.max() > 64 and len(corners) > 1
    gpu = run_gpu(sites, dom, want_grad=grad)
    assert gpu["info"]["status"] == 0
    assert_parity(gpu, ref, oracle_mod.site_moments(ref, sites), len(sites))
    site, simp = gpu["res"]["piece_site"], gpu["res"]["piece_simplex"]
    assert len(np.unique(site * dom.m + simp)) == len(site)


def _many():
    """Cells of 40 faces, which leave the sweep whole, and those of CUT, halfway."""
    grid = (np.stack(np.meshgrid(*[np.arange(3)] * 3), -1).reshape(-1, 3) + 0.5) / 3
    out = []
    for i, at in enumerate(grid):
        seed, radius, _ = CUT[i % len(CUT)]
        b = _ball(40 if i % 2 else 33, seed + i, 0.3 * radius, at)
        out.append(b + 1e-6 * np.random.default_rng(i).standard_normal(b.shape))
    return np.vstack(out), vdgen.kuhn_cube_grid(6, jitter=0.1, seed=1)


def test_no_sync_with_a_list():
    import torch
    import paper_2509_07175_amd as vd
    host, mesh = _many()
    n = len(host)
    dom = vd.Domain.from_vdgen(mesh)
    box = (0.0, 0.0, 0.0, 1.0, 1.0, 1.0)
    sites = torch.as_tensor(host, device="cuda")
    grid, cells = vd.Grid(), vd.Cells()
    opts = dict(want_grad=1)
    side = torch.cuda.Stream()
    out = [torch.empty(s, dtype=torch.float64, device="cuda") for s in ((n,), (n, 3), (n,))]
    with torch.cuda.stream(side):
        vd.build_grid(sites, bbox=box, grid=grid)
        vd.clip_cells(grid, dom, vd.Options.default(**opts), cells=cells)
    torch.cuda.synchronize()
    ref = [t.clone() for t in cells.moments()]
    vd.clip_cells(grid, dom, vd.Options.default(no_sync=1, **opts), cells=cells)
    got = cells.moments()
    torch.cuda.synchronize()
    assert cells.info()["status"] == 0
    assert all(torch.equal(a, b) for a, b in zip(ref, got))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        vd.build_grid(sites, bbox=box, grid=grid)
        vd.clip_cells(grid, dom, vd.Options.default(no_sync=1, **opts), cells=cells)
        cells.moments(*out)
    for rep in range(3):
        sites.copy_(torch.as_tensor(host + 1e-6 * np.random.default_rng(rep).standard_normal(host.shape)))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert cells.info()["status"] == 0
        eager = vd.clip_cells(vd.build_grid(sites.clone(), bbox=box), dom, vd.Options.default(**opts))
        want = eager.moments()
        torch.cuda.synchronize()
        log(f"replay {rep}: pieces {cells.info()['n_pieces']} eager {eager.info()['n_pieces']}")
        assert cells.info()["n_pieces"] == eager.info()["n_pieces"]
        assert all(torch.equal(a, b) for a, b in zip(out, want))
