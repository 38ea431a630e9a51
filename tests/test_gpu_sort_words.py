"""The radix sort behind the builds and the searches: 32-bit keys (up to four
8-bit passes) and 64-bit ones, at the sizes where its launches change (one
tile of 2,048, up to 96 tiles, more), on clouds whose neighbours share their
top digits and on shuffled ones.  Layouts follow the rules of
``tests/test_gpu_parity.py`` (stable Morton order); the group search, which
sorts its queries, gives the wavefront search's bits.
"""
import numpy as np
import pytest

from paper_2308_07173_amd import workloads
from tests.test_gpu_parity import check_layout

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shuffled", [False, True])
@pytest.mark.parametrize("scale,cell", [(2.0, 1.0), (30.0, 1.0), (900.0, 0.5)])
@pytest.mark.parametrize("n", [2, 2047, 2048, 2049, 196608, 196609, 400001])
def test_sorted_layout_and_queries(n, scale, cell, shuffled):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_07173_amd import lkc
    ctx = lkc.Context()
    p = workloads.random_cloud(n, n + int(scale), scale=scale, offset=(3.0, -7.0, 1.0))
    if not shuffled:
        p = np.ascontiguousarray(p[np.lexsort((p[:, 1], p[:, 0]))])
    d = torch.from_numpy(p).cuda()
    t = lkc.lkc_build_target(ctx, d, cell)
    check_layout(t, p, cell)
    q = d[: min(n, 5000)].contiguous()
    a = lkc.lkc_knn_cov(ctx, t, q, 8, 2 * cell, 1e-3, cfg=dict(algorithm=1))
    b = lkc.lkc_knn_cov(ctx, t, q, 8, 2 * cell, 1e-3, cfg=dict(algorithm=2))
    for key in a:
        assert torch.equal(a[key], b[key]), key
    t.free()
    ctx.close()
