"""Sites on regular lattices, exact and with noise around the rounding of their
coordinates: four and more bisectors meet in a corner, and planes contain edges
of the cell up to rounding.  A clip either refuses such sites (degenerate, or
more faces than it holds) or gives every cell its volume.  The volumes come from
the cell's faces one by one -- the square of each plane cut by all other
half-spaces, times a third of its distance -- which needs no topology, so no
position of the sites is special to it."""
import functools

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


def _lattice(name, noise, seed):
    k = 3 if name in ("fcc", "bcc") else 4
    g = np.stack(np.meshgrid(*[np.arange(k)] * 3), -1).reshape(-1, 3).astype(float)
    if name in ("cubic", "turned"):
        s = (g + 0.5) / k
    elif name == "bcc":
        s = np.vstack([g + 0.25, g + 0.75]) / k
    elif name == "fcc":
        s = np.vstack([g + 0.25 + np.array(d) for d in ([0, 0, 0], [0.5, 0.5, 0], [0.5, 0, 0.5], [0, 0.5, 0.5])]) / k
    else:  # hexagonal layers
        s = np.stack([(g[:, 0] + 0.5 * (g[:, 1] % 2) + 0.25) / k, (g[:, 1] + 0.25) * np.sqrt(0.75) / k,
                      (g[:, 2] + 0.5) / k], 1)
    if name == "turned":
        c, d = np.cos(0.3), np.sin(0.3)
        s = 0.5 + 0.6 * (s - 0.5) @ np.array([[c, -d, 0], [d, c, 0], [0, 0, 1]]).T @ np.array(
            [[1, 0, 0], [0, c, -d], [0, d, c]]).T
    return s + noise * np.random.default_rng(seed).standard_normal(s.shape)


def _volumes(sites):
    """Volumes of the cells in the unit cube."""
    n = len(sites)
    s = sites
    normal = np.zeros((n, n + 6, 3))
    off = np.zeros((n, n + 6))
    d = s[None] - s[:, None]
    r = np.sqrt((d ** 2).sum(-1))
    r[np.arange(n), np.arange(n)] = 1e-3  # (first in order, left out)
    normal[:, :n] = d / r[..., None]
    off[:, :n] = r / 2
    for ax in range(3):
        normal[:, n + 2 * ax, ax], off[:, n + 2 * ax] = -1, s[:, ax]
        normal[:, n + 2 * ax + 1, ax], off[:, n + 2 * ax + 1] = 1, 1 - s[:, ax]
    vol = np.zeros(n)
    for i in range(n):
        # the sites that can carry a face: nearer than twice the cell's radius
        keep = np.concatenate([np.argsort(r[i])[1:51], np.arange(n, n + 6)])
        N, c = normal[i][keep], off[i][keep]
        F = len(keep)
        e = np.where((np.abs(N[:, 0]) < 0.6)[:, None], [[1.0, 0, 0]], [[0, 1.0, 0]])
        a = np.cross(N, e)
        a /= np.sqrt((a ** 2).sum(-1))[:, None]
        b = np.cross(N, a)
        # polygons of all faces at once: m vertices each, the last one repeated
        poly = np.broadcast_to(np.array([[-4, -4], [4, -4], [4, 4], [-4, 4]]), (F, 4, 2)).copy()
        for g in range(F):
            A, B = a @ N[g], b @ N[g]
            C = c[g] - (N @ N[g]) * c
            x = A[:, None] * poly[..., 0] + B[:, None] * poly[..., 1] - C[:, None]
            x[g] = -1  # a plane does not cut its own face
            y = np.roll(x, -1, 1)
            q = np.roll(poly, -1, 1)
            with np.errstate(all="ignore"):
                t = (x / (x - y))[..., None]
                cross = poly + t * (q - poly)
            new = np.stack([poly, cross], 2).reshape(F, -1, 2)
            use = np.stack([x <= 0, (x <= 0) != (y <= 0)], 2).reshape(F, -1)
            cnt = use.sum(1)
            m = max(int(cnt.max()), 1)
            order = np.argsort(~use, 1, kind="stable")[:, :m]
            poly = np.take_along_axis(new, order[..., None], 1)
            last = np.maximum(cnt - 1, 0)
            pad = np.arange(m)[None] > last[:, None]
            poly = np.where(pad[..., None], poly[np.arange(F), last][:, None], poly)
            poly[cnt == 0] = 0
        x, y = poly[..., 0], poly[..., 1]
        x, y = x - x[:, :1], y - y[:, :1]
        area = 0.5 * (x * np.roll(y, -1, 1) - y * np.roll(x, -1, 1)).sum(1)
        vol[i] = (area * c).sum() / 3
    return vol


@functools.lru_cache(None)
def _case(name, noise):
    sites = _lattice(name, noise, seed=7)
    vol = _volumes(sites)
    assert abs(vol.sum() - 1) < 1e-12
    return sites, vol


@pytest.mark.parametrize("noise", [0.0, 1e-16, 1e-15, 1e-14, 1e-12, 1e-10, 1e-8, 1e-6])
@pytest.mark.parametrize("name", ["cubic", "bcc", "fcc", "hexagonal", "turned"])
def test_lattice_cells(name, noise):
    import torch
    import paper_2509_07175_amd as vd
    sites, vol = _case(name, noise)
    for dom in (vdgen.kuhn_cube_grid(1), vdgen.kuhn_cube_grid(2, jitter=0.1, seed=3)):
        s = torch.as_tensor(sites, dtype=torch.float64, device="cuda")
        d = vd.Domain.from_vdgen(dom)
        g = vd.build_grid(s, bbox=(0.0, 0.0, 0.0, 1.0, 1.0, 1.0))
        # (equal weights: the same cells as a power diagram)
        w = vd.build_grid(s, bbox=(0.0, 0.0, 0.0, 1.0, 1.0, 1.0), weights=torch.full((len(sites),), 0.25, device="cuda", dtype=torch.float64))
        for grid, opts in ((g, {}), (g, {"want_grad": 1}), (g, {"whole_interior": 1}), (w, {}), (g, {"improved_search": 1})):
            try:
                c = vd.clip_cells(grid, d, vd.Options.default(**opts))
            except vd.VDError as e:
                log(f"{name} noise {noise} m={dom.m} {opts}: {e}")
                assert e.status in (4, 5) and noise < 1e-12
                continue
            m, _, _ = c.moments()
            err = np.abs(m.cpu().numpy() - vol) / vol
            log(f"{name} noise {noise} m={dom.m} {opts}: {err.max():.1e}")
            assert err.max() < 1e-9
