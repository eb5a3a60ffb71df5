"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is one pass through the public entry points: grid build, clip and moments (and the adjoint, Lloyd steps, a
batch in a graph) on sites that are already on the GPU, for a staged domain, with the handles that a program keeps
between passes.  Outputs are the per-site moments, gradients, moved sites, and for one case the lists of the diagram.

  cells     grid + clip + moments in a cube of Kuhn tetrahedra (uniform or clustered sites)
  grad      the same with face moments, and the adjoint of a loss on mass, centroid and energy
  autograd  VoronoiMoments.apply and loss.backward(), as in a training loop
  diagram   grid + clip on a non-convex L-shaped block, and the diagram's lists (pieces, neighbours)
  lloyd     lloyd(): some iterations with a quadratic density, or with whole interior cells
  sphere    restricted diagram on a triangulated sphere, forward
  sphere_grad   ... and with the adjoint
  batch     many small diagrams of uneven size as one batch, captured in a graph and replayed
  power     a power diagram (weighted sites), forward
"""
import functools
import itertools
import math

import numpy as np
import torch

import paper_2509_07175_amd as vd

UNIT = (0.0, 0.0, 0.0, 1.0, 1.0, 1.0)
BALL = (-1.01, -1.01, -1.01, 1.01, 1.01, 1.01)
DENSITY = (1.0, 0.5, -0.3, 0.2, 0.4, 0.1, -0.2, 0.3, 0.05, 0.6)  # positive on the unit cube
DEV = "cuda" if torch.cuda.is_available() else "cpu"


def listed():
    return [
        # a small clipped diagram, as in an inner loop over many of them: launches and waits count
        {"name": "cube_1k", "kind": "cells", "n": 1000, "k": 1, "sites": "uniform"},
        # a simulation step on a medium mesh: cells and mesh elements alike in size
        {"name": "mesh_100k", "kind": "cells", "n": 100_000, "k": 20, "sites": "uniform"},
        # adaptive sampling: sites concentrated where the detail is, a fine mesh (the headline workload)
        {"name": "clustered_1m", "kind": "cells", "n": 1_000_000, "k": 50, "sites": "clustered"},
        # white noise in a box, the largest call
        {"name": "cube_5m", "kind": "cells", "n": 5_000_000, "k": 1, "sites": "uniform"},
        # one step of an optimisation over the sites, handles kept by the program
        {"name": "clustered_grad", "kind": "grad", "n": 200_003, "k": 30, "sites": "clustered"},
        # a training step through torch.autograd
        {"name": "autograd_4k", "kind": "autograd", "n": 4099, "k": 6, "sites": "uniform"},
        # meshing a non-convex part: the incidence and neighbour lists are the result
        {"name": "diagram_l_20k", "kind": "diagram", "n": 20_011, "k": 12, "sites": "uniform"},
        # density-weighted centroidal tessellation
        {"name": "lloyd_60k", "kind": "lloyd", "n": 60_000, "k": 16, "iters": 4, "density": True, "whole": False},
        # remeshing a surface: restricted diagram and gradient
        {"name": "sphere_200k", "kind": "sphere_grad", "n": 200_000, "level": 6},
        # the same on a coarse mesh, forward only
        {"name": "sphere_3k", "kind": "sphere", "n": 3001, "level": 3},
        # many independent diagrams at once
        {"name": "batch_48", "kind": "batch", "num": 48, "lo": 1000, "hi": 16_000, "klo": 6, "khi": 16, "layout": 105},
        # weighted sites
        {"name": "power_30k", "kind": "power", "n": 30_000, "k": 10},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["cells", "cells", "cells", "grad", "autograd", "diagram", "lloyd", "sphere", "sphere_grad",
                       "batch", "power"])
    if kind in ("cells", "grad"):
        n = _log(rng, 100, 2_000_000 if kind == "cells" else 600_000)
        # from one cube of six tetrahedra to about as many tetrahedra as sites
        k = _log(rng, 1, max(1.01, min(50.0, 1.2 * (n / 6.0) ** (1.0 / 3.0))))
        return {"kind": kind, "n": n, "k": k, "sites": rng.choice(["uniform", "clustered"])}
    if kind == "autograd":
        return {"kind": kind, "n": _log(rng, 200, 60_000), "k": rng.randint(1, 12), "sites": rng.choice(["uniform", "clustered"])}
    if kind == "diagram":
        return {"kind": kind, "n": _log(rng, 500, 100_000), "k": 2 * rng.randint(2, 10), "sites": "uniform"}
    if kind == "lloyd":
        whole = rng.random() < 0.5
        return {"kind": kind, "n": _log(rng, 1000, 150_000), "k": rng.randint(1, 20), "iters": rng.randint(2, 6),
                "density": not whole, "whole": whole}
    if kind in ("sphere", "sphere_grad"):
        level = rng.randint(2, 6)
        return {"kind": kind, "n": _log(rng, 300, min(400_000, 24 * 20 * 4 ** level)), "level": level}
    if kind == "batch":
        return {"kind": kind, "num": rng.randint(8, 96), "lo": rng.randint(100, 1000), "hi": rng.randint(2000, 12_000),
                "klo": rng.randint(2, 6), "khi": rng.randint(7, 12), "layout": rng.randrange(1 << 20)}
    return {"kind": kind, "n": _log(rng, 300, 60_000), "k": rng.randint(1, 12)}


# ---- inputs -------------------------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 1_000_003 + 17)


def _cube_sites(n, how, g):
    s = torch.rand((n, 3), dtype=torch.float64, device=DEV, generator=g)
    if how == "clustered":  # 8 Gaussians of sigma 0.05 and 10 % of uniform background
        c = 0.2 + 0.6 * torch.rand((8, 3), dtype=torch.float64, device=DEV, generator=g)
        which = torch.randint(0, 8, (n,), device=DEV, generator=g)
        p = c[which] + 0.05 * torch.randn((n, 3), dtype=torch.float64, device=DEV, generator=g)
        keep = ((p > 0) & (p < 1)).all(1) & (torch.rand(n, dtype=torch.float64, device=DEV, generator=g) < 0.9)
        s = torch.where(keep[:, None], p, s)
    return s.clamp(1e-9, 1 - 1e-9).contiguous()


def _l_sites(n, g):
    """Uniform in the unit cube without its quarter x, y > 1/2."""
    s = torch.rand((n, 3), dtype=torch.float64, device=DEV, generator=g).clamp(1e-9, 1 - 1e-9)
    part = torch.randint(0, 3, (n,), device=DEV, generator=g)
    s[:, 0] = 0.5 * s[:, 0] + 0.5 * (part == 1)
    s[:, 1] = 0.5 * s[:, 1] + 0.5 * (part == 2)
    return s.contiguous()


def _sphere_sites(n, g):
    p = torch.randn((n, 3), dtype=torch.float64, device=DEV, generator=g)
    return (p / p.norm(dim=1, keepdim=True)).contiguous()


@functools.lru_cache(maxsize=None)
def _kuhn(k, shape="cube"):
    """k^3 cubes of the unit cube, six Kuhn tetrahedra each; shape "l": without the cubes of the quarter x, y > 1/2."""
    n1 = k + 1
    z, y, x = np.meshgrid(np.arange(n1), np.arange(n1), np.arange(n1), indexing="ij")
    verts = np.stack([x.ravel(), y.ravel(), z.ravel()], axis=1) / k
    cz, cy, cx = np.meshgrid(np.arange(k), np.arange(k), np.arange(k), indexing="ij")
    c = np.stack([cx.ravel(), cy.ravel(), cz.ravel()], axis=1)
    if shape == "l":
        c = c[(c[:, 0] < k // 2) | (c[:, 1] < k // 2)]
    tets = []
    for perm in itertools.permutations(range(3)):
        p = [c]
        for ax in perm:
            q = p[-1].copy()
            q[:, ax] += 1
            p.append(q)
        ids = np.stack([q[:, 0] + n1 * (q[:, 1] + n1 * q[:, 2]) for q in p], axis=1)
        if np.linalg.det(np.eye(3)[list(perm)]) < 0:
            ids = ids[:, [0, 1, 3, 2]]
        tets.append(ids)
    tets = np.stack(tets, axis=1).reshape(-1, 4)
    used, tets = np.unique(tets, return_inverse=True)
    return verts[used], tets.reshape(-1, 4).astype(np.int32)


@functools.lru_cache(maxsize=None)
def _icosphere(level):
    t = (1.0 + 5.0 ** 0.5) / 2.0
    v = np.array([[-1, t, 0], [1, t, 0], [-1, -t, 0], [1, -t, 0], [0, -1, t], [0, 1, t], [0, -1, -t], [0, 1, -t],
                  [t, 0, -1], [t, 0, 1], [-t, 0, -1], [-t, 0, 1]], dtype=np.float64)
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    f = np.array([[0, 11, 5], [0, 5, 1], [0, 1, 7], [0, 7, 10], [0, 10, 11], [1, 5, 9], [5, 11, 4], [11, 10, 2],
                  [10, 7, 6], [7, 1, 8], [3, 9, 4], [3, 4, 2], [3, 2, 6], [3, 6, 8], [3, 8, 9], [4, 9, 5], [2, 4, 11],
                  [6, 2, 10], [8, 6, 7], [9, 8, 1]], dtype=np.int64)
    for _ in range(level):
        e = np.sort(np.stack([f[:, [0, 1]], f[:, [1, 2]], f[:, [2, 0]]], axis=1).reshape(-1, 2), axis=1)
        uniq, inv = np.unique(e, axis=0, return_inverse=True)
        mid = v[uniq].mean(axis=1)
        mid /= np.linalg.norm(mid, axis=1, keepdims=True)
        m = inv.reshape(-1, 3) + len(v)
        v = np.concatenate([v, mid])
        f = np.concatenate([np.stack(q, axis=1) for q in (
            (f[:, 0], m[:, 0], m[:, 2]), (f[:, 1], m[:, 1], m[:, 0]), (f[:, 2], m[:, 2], m[:, 1]),
            (m[:, 0], m[:, 1], m[:, 2]))])
    q = v[f]
    inward = np.einsum("ij,ij->i", np.cross(q[:, 1] - q[:, 0], q[:, 2] - q[:, 0]), q.mean(axis=1)) < 0
    f[inward] = f[inward][:, [0, 2, 1]]
    return v, f.astype(np.int32)


def _area(level):
    v, f = _icosphere(level)
    q = v[f]
    return float(0.5 * np.linalg.norm(np.cross(q[:, 1] - q[:, 0], q[:, 2] - q[:, 0]), axis=1).sum())


def _mesh_of(case):
    if case["kind"].startswith("sphere"):
        return _icosphere(case["level"]) + (2,)
    return _kuhn(case["k"], "l" if case["kind"] == "diagram" else "cube") + (3,)


def _batch_layout(case):
    """Site counts (log-uniform) and mesh sizes of a batch: what a program knows before it has the sites."""
    r = np.random.default_rng(case["layout"])
    n = np.exp(r.uniform(np.log(case["lo"]), np.log(case["hi"]), case["num"])).round().astype(int)
    k = r.integers(case["klo"], case["khi"] + 1, case["num"])
    return [int(x) for x in n], [int(x) for x in k]


def _inputs(case, seed):
    """The tensors of a case: sites, weights and upstream gradients."""
    g = _gen(seed)
    kind = case["kind"]
    d = {}
    if kind == "batch":
        d["sites"] = _cube_sites(sum(_batch_layout(case)[0]), "uniform", g)
        return d
    n = case["n"]
    if kind.startswith("sphere"):
        d["sites"] = _sphere_sites(n, g)
    elif kind == "diagram":
        d["sites"] = _l_sites(n, g)
    else:
        d["sites"] = _cube_sites(n, case.get("sites", "uniform"), g)
    if kind == "power":  # about the square of the distance between sites times n^(-1/3)
        d["weights"] = (2 * torch.rand(n, dtype=torch.float64, device=DEV, generator=g) - 1) / n
    if kind in ("grad", "autograd", "sphere_grad"):
        d["gm"] = torch.randn(n, dtype=torch.float64, device=DEV, generator=g)
        d["gc"] = torch.randn((n, 3), dtype=torch.float64, device=DEV, generator=g)
        d["ge"] = 1 + torch.rand(n, dtype=torch.float64, device=DEV, generator=g)
    return d


def _domain(verts, simplices, dim):
    return vd.Domain(torch.as_tensor(verts, dtype=torch.float64, device=DEV).contiguous(),
                     torch.as_tensor(simplices, dtype=torch.int32, device=DEV).contiguous(), None, dim)


def _sites_per_cell(case):
    return 0.25 if case.get("sites") == "clustered" else 0.0  # a finer grid where sites are dense in places


def _out(n):
    e = functools.partial(torch.empty, dtype=torch.float64, device=DEV)
    return {"mass": e(n), "centroid": e((n, 3)), "energy": e(n), "grad": e((n, 3))}


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, **_inputs(case, seed)}
    n = s["sites"].shape[0]
    if kind != "batch":
        s["domain"] = _domain(*_mesh_of(case))
    if kind in ("cells", "grad", "diagram", "sphere", "sphere_grad", "power"):
        s.update(grid=vd.Grid(), cells=vd.Cells(), **_out(n))
        s["options"] = vd.Options.default(want_grad=1 if "gm" in s else 0)
        s["area"] = _area(case["level"]) if kind.startswith("sphere") else 0.0
        if kind == "diagram":
            s["simplex"], s["nbr"] = (torch.empty(x, dtype=torch.int32, device=DEV) for x in (16 * n + 12 * s["domain"].m, 40 * n))
    elif kind == "autograd":
        s["options"] = vd.Options.default(want_grad=1)
    elif kind == "lloyd":
        s["options"] = vd.Options.default(whole_interior=1 if case["whole"] else 0, **({"density": DENSITY} if case["density"] else {}))
    else:
        _prepare_batch(s, case)
    return s


def _prepare_batch(s, case):
    """The batch sized by a first pass, then captured: a serving program does this once per layout."""
    ns, ks = _batch_layout(case)
    meshes = [_kuhn(k) for k in ks]
    so, vo, mo = [0], [0], [0]
    for n, (v, t) in zip(ns, meshes):
        so.append(so[-1] + n)
        vo.append(vo[-1] + len(v))
        mo.append(mo[-1] + len(t))
    verts = torch.as_tensor(np.concatenate([v for v, _ in meshes]), dtype=torch.float64, device=DEV)
    tets = torch.as_tensor(np.concatenate([t for _, t in meshes]), dtype=torch.int32, device=DEV)
    s.update(domain=vd.Domain.batch(verts, tets, None, vo, mo, 3), grid=vd.Grid(), cells=vd.Cells(), **_out(so[-1]))
    boxes = [UNIT] * len(ns)

    def work(no_sync):
        vd.build_grid_batch(s["sites"], so, bboxes=boxes, grid=s["grid"])
        vd.clip_cells(s["grid"], s["domain"], vd.Options.default(no_sync=no_sync), cells=s["cells"])
        s["cells"].moments(s["mass"], s["centroid"], s["energy"])

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        work(0)
    torch.cuda.synchronize()
    s["graph"] = torch.cuda.CUDAGraph()
    with torch.cuda.graph(s["graph"]):
        work(1)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "batch":
        s["graph"].replay()
        return s["mass"], s["centroid"], s["energy"]
    if kind == "lloyd":
        return vd.lloyd(s["sites"].clone(), s["domain"], case["iters"], options=s["options"], bbox=UNIT)
    if kind == "autograd":
        x = s["sites"].clone().requires_grad_(True)
        m, c, e = vd.VoronoiMoments.apply(x, s["domain"], s["options"], UNIT)
        loss = (s["gm"] * m).sum() + (s["gc"] * c).sum() + (s["ge"] * e).sum()
        loss.backward()
        return m.detach(), c.detach(), e.detach(), x.grad
    vd.build_grid(s["sites"], bbox=BALL if kind.startswith("sphere") else UNIT, sites_per_cell=_sites_per_cell(case),
                  surface_area=s["area"], grid=s["grid"], weights=s.get("weights"))
    vd.clip_cells(s["grid"], s["domain"], s["options"], cells=s["cells"])
    s["cells"].moments(s["mass"], s["centroid"], s["energy"])
    out = [s["mass"], s["centroid"], s["energy"]]
    if kind == "diagram":
        v = s["cells"].view()  # the lists go to buffers that hold the next steps' diagrams too, -1 behind their ends
        ids = v["piece_id"].long()
        for buf, x in ((s["simplex"], v["piece_simplex"][ids]), (s["nbr"], v["nbr"])):
            buf.fill_(-1)
            buf[:len(x)] = x
        out += [v["cell_piece_off"], s["simplex"], v["nbr_off"], s["nbr"]]
    if "gm" in s:
        out.append(s["cells"].backward(s["gm"], s["gc"], s["ge"], out=s["grad"]))
    return out


def work(case):
    """Bytes: the sites and the mesh read once, the returned values (and the emitted polytopes) written once.
    Operations: a Poisson-Voronoi cell has 27 corners (a 3x3 solve, 51 flops, each) and three fan tetrahedra (78 flops)
    per corner; a restricted cell about 6 corners of 51 flops and as many fan triangles of 30."""
    if case["kind"] == "batch":
        ns, ks = _batch_layout(case)
        parts = [(n, 8 * (k + 1) ** 3 * 3 + 6 * k ** 3 * 32) for n, k in zip(ns, ks)]
        return {"bytes": float(sum(n * (24 + 40 + 27 * 36 + 16 * 4) + m for n, m in parts)), "flops": float(sum(n for n, _ in parts) * 27 * (51 + 234))}
    n = case["n"]
    verts, simp, dim = _mesh_of(case)
    mesh = verts.nbytes + 2 * simp.nbytes
    grad = "grad" in case["kind"]
    per = 24 + 40 + (27 * 36 + 16 * 4 if dim == 3 else 6 * 40) + (64 if grad else 0)
    flops = 27 * (51 + 234) if dim == 3 else 6 * 81
    if grad:
        flops += 15.5 * 5.2 * 60 if dim == 3 else 6 * 60
    it = case.get("iters", 1)
    return {"bytes": float(it * (n * per + mesh)), "flops": float(it * n * flops)}


# ---- the same in plain torch: every face of a cell is a polygon on a bisector (or on a side of the domain), clipped by
# ---- the other bisectors; moments from the cones over the faces, gradients from the faces' integrals.  Float64.

def _clip(p, cnt, nrm, off):
    """Convex polygons p [B, V, 3] of cnt corners clipped by nrm.x <= off (one half-space each)."""
    B, V, _ = p.shape
    j = torch.arange(V, device=p.device)[None]
    live = j < cnt[:, None]
    d = (p * nrm[:, None]).sum(2) - off[:, None]
    ins = (d <= 0) & live
    nxt = torch.where(j + 1 < cnt[:, None], j + 1, torch.zeros_like(j))
    dn, pn, inn = d.gather(1, nxt), p.gather(1, nxt[..., None].expand(-1, -1, 3)), ins.gather(1, nxt)
    cross = (ins != inn) & live
    x = p + (pn - p) * (d / (d - dn + (d == dn)))[..., None]
    e = ins.long() + cross.long()
    at = e.cumsum(1) - e
    total = e.sum(1)
    out = torch.zeros((B, V + 1, 3), dtype=p.dtype, device=p.device)
    spare = torch.full_like(at, V)
    out.scatter_(1, torch.where(ins, at, spare)[..., None].expand(-1, -1, 3), p)
    out2 = torch.zeros_like(out)
    out2.scatter_(1, torch.where(cross, at + ins.long(), spare)[..., None].expand(-1, -1, 3), x)
    mark = torch.zeros((B, V + 1), dtype=torch.bool, device=p.device).scatter_(1, torch.where(cross, at + ins.long(), spare), True)
    assert int(total.max()) < V
    return torch.where(mark[..., None], out2, out)[:, :V].contiguous(), total


def _fan(p, cnt):
    """Triangles (first corner, corner, next) of each polygon: index of the polygon, corners [T, 3, 3]."""
    V = p.shape[1]
    j = torch.arange(1, V - 1, device=p.device)[None]
    b, k = torch.nonzero(j + 1 < cnt[:, None], as_tuple=True)
    return b, torch.stack([p[b, 0], p[b, k + 1], p[b, k + 2]], 1)


def _near(v, K):
    n = v.shape[0]
    idx, dist = [], []
    for a in range(0, n, 1024):
        d = torch.zeros((min(1024, n - a), n), dtype=v.dtype, device=v.device)
        for c in range(3):
            d += (v[a:a + 1024, None, c] - v[None, :, c]) ** 2
        q = d.topk(K + 1, largest=False)
        idx.append(q.indices[:, 1:])
        dist.append(q.values[:, 1:].sqrt())
    return torch.cat(idx), torch.cat(dist)


def _cells_exact(v, boxes, w, rho, grads):
    """(mass, centroid, energy, gradient) of the cells of v in a union of boxes, or None if they reach too far."""
    n = v.shape[0]
    K = min(n - 1, 200)
    nb, dist = _near(v, K)
    w = torch.zeros(n, dtype=v.dtype, device=v.device) if w is None else w
    faces, reach = [], torch.zeros(n, dtype=v.dtype, device=v.device)
    step = 2000
    for box in boxes:
        lo, hi = (torch.tensor(x, dtype=v.dtype, device=v.device) for x in (box[:3], box[3:]))
        for a in range(0, n, step):
            i = torch.arange(a, min(n, a + step), device=v.device)
            m = len(i)
            bn = v[nb[i]] - v[i, None]
            bo = 0.5 * ((bn ** 2).sum(2) + w[i, None] - w[nb[i]])
            eye = torch.eye(3, dtype=v.dtype, device=v.device)
            N = torch.cat([bn, eye.expand(m, 3, 3), -eye.expand(m, 3, 3)], 1)
            O = torch.cat([bo, hi - v[i], v[i] - lo], 1)
            F = K + 6
            own, f = (t.reshape(-1) for t in torch.meshgrid(torch.arange(m, device=v.device), torch.arange(F, device=v.device), indexing="ij"))
            fn, fo = N[own, f], O[own, f]
            ln = fn.norm(dim=1, keepdim=True)
            u = fn / ln
            t1 = torch.linalg.cross(u, torch.where(u[:, :1].abs() < 0.6, eye[0], eye[1]).expand_as(u))
            t1 = t1 / t1.norm(dim=1, keepdim=True)
            t2 = torch.linalg.cross(u, t1)
            c0 = u * (fo[:, None] / ln)
            p = torch.stack([c0 + 4 * (x * t1 + y * t2) for x, y in ((1, 1), (-1, 1), (-1, -1), (1, -1))], 1)
            p = torch.cat([p, torch.zeros((len(p), 28, 3), dtype=v.dtype, device=v.device)], 1)
            cnt = torch.full((len(p),), 4, device=v.device)
            for h in itertools.chain(range(K, F), range(K)):
                same = f == h
                q, c = _clip(p, cnt, N[own, h], O[own, h])
                p = torch.where(same[:, None, None], p, q)
                cnt = torch.where(same, cnt, c)
                keep = torch.nonzero(cnt >= 3).squeeze(1)
                if len(keep) < 0.9 * len(p):
                    p, cnt, own, f = p[keep], cnt[keep], own[keep], f[keep]
            keep = torch.nonzero(cnt >= 3).squeeze(1)
            p, cnt, own, f = p[keep], cnt[keep], own[keep], f[keep]
            far = (p.norm(dim=2) * (torch.arange(p.shape[1], device=v.device)[None] < cnt[:, None])).amax(1)
            reach.scatter_reduce_(0, i[own], far, "amax")
            faces.append((i[own], torch.where(f < K, nb[i[own], f.clamp(max=K - 1)], -1), p[:, :20], cnt))
    if K < n - 1 and bool((reach + (reach ** 2 + (w.max() - w).clamp(min=0)).sqrt() > dist[:, -1]).any()):
        return None
    return _sum_faces(v, w, faces, rho, grads)


def _duffy(dim):
    """Points and weights of the unit simplex's product rule (four Gauss points a direction: exact far beyond need)."""
    x, wt = np.polynomial.legendre.leggauss(4)
    x, wt = 0.5 * (x + 1), 0.5 * wt
    pts, ws = [], []
    for q in itertools.product(range(4), repeat=dim):
        rest, bary, wq = 1.0, [], 1.0
        for lev, a in enumerate(q):
            wq *= wt[a] * (1 - x[a]) ** (dim - 1 - lev)
            bary.append(rest * x[a])
            rest *= 1 - x[a]
        pts.append([rest] + bary)
        ws.append(wq * math.factorial(dim))
    return np.array(pts), np.array(ws)


def _rho_at(x, rho):
    if rho is None:
        return torch.ones(x.shape[:-1], dtype=x.dtype, device=x.device)
    a, b, c = x.unbind(-1)
    return (rho[0] + rho[1] * a + rho[2] * b + rho[3] * c + rho[4] * a * a + rho[5] * a * b + rho[6] * a * c +
            rho[7] * b * b + rho[8] * b * c + rho[9] * c * c)


def _sum_faces(v, w, faces, rho, grads):
    n = v.shape[0]
    M = torch.zeros(n, dtype=v.dtype, device=v.device)
    C, E = torch.zeros_like(v), torch.zeros_like(M)
    pts, ws = (torch.tensor(t, dtype=v.dtype, device=v.device) for t in _duffy(3))
    tri = []
    for own, other, p, cnt in faces:
        b, t = _fan(p, cnt)
        o, k = own[b], other[b]
        vol = (t[:, 0] * torch.linalg.cross(t[:, 1], t[:, 2])).sum(1) / 6  # signed: a power cell need not hold its site
        for a in range(0, len(t), 200_000):
            s = slice(a, a + 200_000)
            x = torch.einsum("qk,tkc->tqc", pts[:, 1:], t[s])
            q = _rho_at(x + v[o[s], None], rho) * ws * vol[s, None]
            M.index_add_(0, o[s], q.sum(1))
            C.index_add_(0, o[s], (q[..., None] * x).sum(1))
            E.index_add_(0, o[s], (q * (x ** 2).sum(2)).sum(1))
        tri.append((o, k, t))
    hit = M > 0
    cen = torch.where(hit[:, None], v + C / torch.where(hit, M, torch.ones_like(M))[:, None], v)
    if grads is None:
        return M, cen, E, None
    gm, gc, ge = grads
    b_ = gc / M[:, None]
    a_ = gm - (b_ * cen).sum(1)
    G = 2 * ge[:, None] * M[:, None] * (v - cen)
    pts, ws = (torch.tensor(t, dtype=v.dtype, device=v.device) for t in _duffy(2))
    for o, k, t in tri:
        on = k >= 0
        o, k, t = o[on], k[on], t[on]
        area = 0.5 * torch.linalg.cross(t[:, 1] - t[:, 0], t[:, 2] - t[:, 0]).norm(dim=1)
        x = torch.einsum("qk,tkc->tqc", pts, t)
        f = (a_[o] - a_[k])[:, None] + ((b_[o] - b_[k])[:, None] * (x + v[o, None])).sum(2) + (ge[o] - ge[k])[:, None] * (x ** 2).sum(2)
        f = f * _rho_at(x + v[o, None], rho) * ws * (area / (v[k] - v[o]).norm(dim=1))[:, None]
        G.index_add_(0, o, (f[..., None] * x).sum(1))
    return M, cen, E, G


def _sphere_exact(v, verts, tris, grads):
    n, m = v.shape[0], len(tris)
    q = torch.as_tensor(verts, dtype=v.dtype, device=v.device)[torch.as_tensor(tris.astype(np.int64), device=v.device)]
    cen = q.mean(1)
    rad = (q - cen[:, None]).norm(dim=2).amax(1)
    pairs = []
    for a in range(0, m, 512):  # sites that can be nearest to a point of the triangle
        d = (cen[a:a + 512, None] - v[None]).norm(dim=2)
        near = d.amin(1)
        t, s = torch.nonzero(d <= near[:, None] + 2 * rad[a:a + 512, None] + 1e-9, as_tuple=True)
        pairs.append((t + a, s))
    t, s = torch.cat([x for x, _ in pairs]), torch.cat([x for _, x in pairs])
    count = torch.bincount(t, minlength=m)
    start = count.cumsum(0) - count
    if float((count.double() ** 2).sum()) > 4e8:
        return None
    p = torch.cat([q[t] - v[s, None], torch.zeros((len(t), 25, 3), dtype=v.dtype, device=v.device)], 1)
    cnt = torch.full((len(t),), 3, device=v.device)
    tag = -torch.ones((len(t), p.shape[1]), dtype=torch.long, device=v.device)
    cand = s
    for h in range(int(count.max())):
        go = h < count[t]
        k = cand[(start[t] + h).clamp(max=len(cand) - 1)]
        go &= k != s
        nrm = v[k] - v[s]
        off = torch.where(go, 0.5 * (nrm ** 2).sum(1), torch.full_like(nrm[:, 0], 1e9))
        p, cnt = _clip(p, cnt, nrm, off)
        keep = torch.nonzero(cnt >= 3).squeeze(1)
        if len(keep) < 0.9 * len(p):
            p, cnt, t, s = p[keep], cnt[keep], t[keep], s[keep]
    keep = torch.nonzero(cnt >= 3).squeeze(1)
    p, cnt, t, s = p[keep], cnt[keep], t[keep], s[keep]
    b, f = _fan(p, cnt)
    o = s[b]
    area = 0.5 * torch.linalg.cross(f[:, 1] - f[:, 0], f[:, 2] - f[:, 0]).norm(dim=1)
    sm = f.sum(1)
    M = torch.zeros(n, dtype=v.dtype, device=v.device).index_add_(0, o, area)
    C = torch.zeros_like(v).index_add_(0, o, area[:, None] * sm / 3)
    E = torch.zeros_like(M).index_add_(0, o, area / 12 * ((f ** 2).sum((1, 2)) + (sm ** 2).sum(1)))
    hit = M > 0
    cen = torch.where(hit[:, None], v + C / torch.where(hit, M, torch.ones_like(M))[:, None], v)
    return [M, cen, E]


def exact(case, seed):
    kind = case["kind"]
    if kind in ("sphere", "sphere_grad"):
        if case["n"] * 20 * 4 ** case["level"] > 2e9:
            return None
        d = _inputs(case, seed)
        verts, tris = _icosphere(case["level"])
        r = _sphere_exact(d["sites"], verts, tris, None)
        return None if r is None else r + ([None] if kind == "sphere_grad" else [])
    if kind == "batch":
        ns, _ = _batch_layout(case)
        if sum(ns) > 30_000 or min(ns) < 2:
            return None
        v, parts = _inputs(case, seed)["sites"], []
        for x in v.split(ns):
            parts.append(_cells_exact(x, [UNIT], None, None, None))
        if any(x is None for x in parts):
            return None
        return [torch.cat([x[j] for x in parts]) for j in range(3)]
    n = case["n"]
    if n > 32_000 * (1 if kind != "lloyd" else 1.0 / case["iters"]):
        return None
    d = _inputs(case, seed)
    v = d["sites"]
    if kind == "lloyd":
        for _ in range(case["iters"]):
            r = _cells_exact(v, [UNIT], None, DENSITY if case["density"] else None, None)
            if r is None:
                return None
            v = r[1]
        return v
    boxes = [(0, 0, 0, 0.5, 1, 1), (0.5, 0, 0, 1, 0.5, 1)] if kind == "diagram" else [UNIT]
    grads = (d["gm"], d["gc"], d["ge"]) if "gm" in d else None
    r = _cells_exact(v, boxes, d.get("weights"), None, grads)
    if r is None:
        return None
    out = list(r[:3])
    if kind == "diagram":
        out += [None] * 4
    if grads is not None:
        out.append(r[3])
    return out
