"""The CSR offsets around the sizes at which their scan changes (one block up to
16,384 elements, 4,096 at a time; tiles of 1,024 beyond), for pieces and
neighbours of cells and of surfaces: exact."""
import numpy as np
import pytest

import vdgen
from gpu_util import assert_csr, assert_neighbour_symmetry, log, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_07175_amd as vd
    vd.load()


@pytest.mark.parametrize("surface", [False, True], ids=["solid", "surface"])
@pytest.mark.parametrize("n", [1, 2, 1024, 4096, 4097, 16384, 16385])
def test_offsets(n, surface):
    log(f"offsets: n={n} surface={surface}")
    if surface:
        dom = vdgen.icosphere(4)
        q = dom.verts[dom.simplices]
        area = 0.5 * np.linalg.norm(np.cross(q[:, 1] - q[:, 0], q[:, 2] - q[:, 0]), axis=1).sum()
        gpu = run_gpu(vdgen.sphere_sites(n, seed=n), dom, bbox=(-1.01, -1.01, -1.01, 1.01, 1.01, 1.01),
                      surface_area=float(area))
        total = float(area)
    else:
        gpu = run_gpu(vdgen.uniform_cube_sites(n, seed=n, jitter=1e-7), vdgen.kuhn_cube_grid(2))
        total = 1.0
    assert gpu["info"]["status"] == 0
    assert_csr(gpu, n)
    assert_neighbour_symmetry(gpu["nbr_off"], gpu["nbr"])
    for i in (0, n // 2, n - 1):
        a, b = gpu["nbr_off"][i:i + 2]
        assert np.all(np.diff(gpu["nbr"][a:b]) > 0)
    assert abs(gpu["mass"].sum() - total) <= 1e-11 * total
