"""Handles made and freed one after another, on several streams and threads:
their blocks go from one to the next, the results stay those of a handle of
their own, and the memory is given back with the last handle."""
import gc
import threading

import pytest

import vdgen
from gpu_util import log

pytestmark = pytest.mark.gpu

SIZES = (300, 4000, 301, 20000, 4000)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_07175_amd as vd
    vd.load()


def _once(n, dom):
    import torch
    import paper_2509_07175_amd as vd
    x = torch.as_tensor(vdgen.uniform_cube_sites(n, seed=n, jitter=1e-7), device="cuda").requires_grad_(True)
    m, c, e = vd.VoronoiMoments.apply(x, dom, None, (0, 0, 0, 1, 1, 1))
    (m.sum() + 2.0 * c.sum() + 3.0 * e.sum()).backward()
    return [t.detach().clone() for t in (m, c, e, x.grad)]


def test_blocks_go_from_handle_to_handle():
    import torch
    import paper_2509_07175_amd as vd
    torch.cuda.synchronize()
    dom = vd.Domain.from_vdgen(vdgen.kuhn_cube_grid(4))
    ref = {}
    for n in SIZES:
        got = _once(n, dom)
        for a, b in zip(ref.setdefault(n, got), got):
            assert torch.equal(a, b)
    bad = []

    def work(k):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            for n in SIZES[k:] + SIZES[:k]:
                got = _once(n, dom)
                st.synchronize()
                if not all(torch.equal(a, b) for a, b in zip(ref[n], got)):
                    bad.append((k, n))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad
    del dom, got
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    dom = vd.Domain.from_vdgen(vdgen.kuhn_cube_grid(4))
    _once(20000, dom)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    kept = before - torch.cuda.mem_get_info()[0]
    del dom
    gc.collect()
    torch.cuda.empty_cache()
    left = before - torch.cuda.mem_get_info()[0]
    log(f"kept between handles {kept >> 20} MiB, after the last one {left >> 20} MiB")
    assert left <= 16 << 20
