"""One GICP linearisation at the sizes where its partial rows change: one
point, the workgroup's edges, 32 rows and one more, the most rows (1,024) and
several points per thread, and either side of the step to the group search,
which reads a transformed copy of the source where the wavefront search moves
each query as it loads it.  The system is the oracle's FP64 reduction of the
correspondences the GPU found (summation order only: the tolerance of
``tests/test_gpu_gicp.py``), and both searches find the same ones.
"""
import numpy as np
import pytest

from oracle import oracle
from paper_2308_07173_amd import workloads
from tests.test_gpu_gicp import check_system

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1, 255, 256, 257, 8192, 8193, 98304, 98305, 300001])
def test_linearize_sizes(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_07173_amd import lkc
    ctx = lkc.Context()
    rng = np.random.default_rng(n)
    tgt = workloads.plane_wall(5000, seed=1)
    src = (tgt[rng.integers(0, 5000, n)] + rng.normal(0, 0.05, (n, 3))).astype(np.float32)

    def covs(m):
        v = rng.normal(size=(m, 3))
        v /= np.linalg.norm(v, axis=1, keepdims=True)
        return (np.eye(3) - 0.999 * v[:, :, None] * v[:, None, :]).astype(np.float32)

    tc, sc = covs(5000), covs(n)
    a = 0.01
    T = np.eye(4)
    T[:2, :2] = [[np.cos(a), -np.sin(a)], [np.sin(a), np.cos(a)]]
    T[:3, 3] = [0.04, -0.03, 0.02]
    d = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    t = lkc.lkc_build_target(ctx, d(tgt), 1.0)
    system, corr = lkc.lkc_gicp_linearize(ctx, t, d(tc), d(src), d(sc), T, 0.5)
    _, other = lkc.lkc_gicp_linearize(ctx, t, d(tc), d(src), d(sc), T, 0.5,
                                      cfg=dict(algorithm=1 if n <= 98304 else 2))
    assert torch.equal(corr, other)
    check_system(lkc.split_system(system),
                 oracle.gicp_linearize(src, sc, tgt, tc, T, corr.cpu().numpy()))
    t.free()
    ctx.close()
