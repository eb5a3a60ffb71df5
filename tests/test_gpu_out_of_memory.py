"""Device memory runs out in the middle of a call: the call reports it, what it
had made is freed, handles that were passed in stay usable, and blocks kept from
freed handles are given back before an allocation fails."""
import gc

import numpy as np
import pytest

import vdgen
from gpu_util import log

pytestmark = pytest.mark.gpu

OUT_OF_MEMORY = 2


@pytest.fixture(autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_07175_amd as vd
    vd.load()
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


def _free():
    import torch
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def _fill(leave):
    """Takes the device's memory but for about `leave` bytes (in steps: large
    blocks leave some behind)."""
    import torch
    out = []
    for _ in range(4):
        n = torch.cuda.mem_get_info()[0] - leave
        if n > 8 << 20:
            out.append(torch.empty(n, dtype=torch.uint8, device="cuda"))
    log(f"left {torch.cuda.mem_get_info()[0]}")
    return out


def _sites(n, seed=1):
    import torch
    return torch.as_tensor(vdgen.uniform_cube_sites(n, seed=seed, jitter=1e-7), device="cuda")


def _mesh(k):
    """A mesh's arrays on the device."""
    import torch
    d = vdgen.kuhn_cube_grid(k)
    return (torch.as_tensor(d.verts, device="cuda"), torch.as_tensor(d.simplices.astype(np.int32), device="cuda"),
            torch.as_tensor(d.adj.astype(np.int32), device="cuda"), 3)


def test_a_domain_that_does_not_fit_leaves_nothing_behind():
    import paper_2509_07175_amd as vd
    dom = vd.Domain.from_vdgen(vdgen.kuhn_cube_grid(2))
    g = vd.build_grid(_sites(2000), bbox=(0, 0, 0, 1, 1, 1))
    vd.clip_cells(g, dom)
    del g, dom
    big = _mesh(80)  # 3 M tetrahedra: 49 MB each of indices and adjacency, and three times that besides
    base = _free()
    filler = _fill(128 << 20)
    with pytest.raises(vd.VDError) as e:
        vd.Domain(*big)
    assert e.value.status == OUT_OF_MEMORY
    del filler, e
    # a handle made and freed: with no other left, the pool is given back as well
    g = vd.build_grid(_sites(200000), bbox=(0, 0, 0, 1, 1, 1))
    del g
    lost = base - _free()
    log(f"lost {lost}")
    assert lost < 4 << 20


def test_a_clip_that_does_not_fit_leaves_its_handles_usable():
    import torch
    import paper_2509_07175_amd as vd
    dom = vd.Domain.from_vdgen(vdgen.kuhn_cube_grid(4))
    small, large = _sites(3000), _sites(1000000, 2)
    grid, cells = vd.Grid(), vd.Cells()
    vd.build_grid(small, bbox=(0, 0, 0, 1, 1, 1), grid=grid)
    ref = [t.clone() for t in vd.clip_cells(grid, dom, cells=cells).moments()]
    filler = _fill(1 << 30)
    vd.build_grid(large, bbox=(0, 0, 0, 1, 1, 1), grid=grid)
    with pytest.raises(vd.VDError) as e:
        vd.clip_cells(grid, dom, cells=cells)
    assert e.value.status == OUT_OF_MEMORY
    del filler, e
    _free()
    vd.build_grid(small, bbox=(0, 0, 0, 1, 1, 1), grid=grid)
    got = vd.clip_cells(grid, dom, cells=cells).moments()
    assert all(torch.equal(a, b) for a, b in zip(ref, got))
    vd.build_grid(large, bbox=(0, 0, 0, 1, 1, 1), grid=grid)
    m, _, _ = vd.clip_cells(grid, dom, cells=cells).moments()
    assert abs(float(m.sum()) - 1.0) < 1e-11


def test_kept_blocks_make_room_for_a_domain():
    import paper_2509_07175_amd as vd
    keep = vd.Domain.from_vdgen(vdgen.kuhn_cube_grid(2))  # a live handle: the pool stays
    g = vd.build_grid(_sites(300000), bbox=(0, 0, 0, 1, 1, 1))
    c = vd.clip_cells(g, keep)
    del g, c
    big = _mesh(80)
    _free()
    filler = _fill(128 << 20)
    d = vd.Domain(*big)  # fits in what the freed handles left
    del filler
    assert abs(d.info()["measure"] - 1.0) < 1e-9
    del d, keep


def test_kept_blocks_are_given_back_on_demand():
    import paper_2509_07175_amd as vd
    keep = vd.Domain.from_vdgen(vdgen.kuhn_cube_grid(2))
    for _ in range(2):  # (the first clip leaves the runtime's scratch memory behind)
        vd.release_memory()
        base = _free()
        g = vd.build_grid(_sites(300000), bbox=(0, 0, 0, 1, 1, 1))
        c = vd.clip_cells(g, keep)
        del g, c
    held = base - _free()
    vd.release_memory()
    left = base - _free()
    log(f"kept {held}, after release {left}")
    assert held > 1 << 28 and left < 4 << 20
    del keep


def test_first_sizes():
    """Faces (4 bytes, 10 a piece) and corners (36 bytes, 16 a piece) take the room of 8
    pieces per site and 3 per simplex also where sites and simplices are alike in
    number and the pieces get more: what a clip with them holds beyond one without."""
    import paper_2509_07175_amd as vd
    dom = vd.Domain.from_vdgen(vdgen.kuhn_cube_grid(22))
    n = 64000
    g = vd.build_grid(_sites(n), bbox=(0, 0, 0, 1, 1, 1))
    used = {}
    for emit in (1, 1, 0):  # (the first clip leaves the runtime's scratch memory behind)
        c = None
        vd.release_memory()
        free = _free()
        c = vd.clip_cells(g, dom, vd.Options.default(emit_polytopes=emit))
        used[emit] = free - _free()
    base = 8 * n + 3 * dom.m + 1024
    log(f"n={n} m={dom.m} {used} {base * (10 * 4 + 16 * 36)}")
    assert used[1] - used[0] < 1.01 * base * (10 * 4 + 16 * 36) + (8 << 20) and c.info()["n_pieces"] > base
