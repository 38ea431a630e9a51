"""The bound with which the wavefront search prunes the rings of a sparse cloud:
the k-th distance itself, not that of some entries more."""
import math
import time

import numpy as np
import pytest

from paper_2308_07173_amd import workloads
from tests import parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

INF = math.inf
WAVE = dict(algorithm=2)


@pytest.fixture(scope="module")
def lk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_07173_amd import lkc
    ctx = lkc.Context()
    yield lkc, ctx
    ctx.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def _ms(*fns):
    """Best times, the calls in turn."""
    best = [INF] * len(fns)
    for _ in range(10):
        for i, fn in enumerate(fns):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            fn()
            torch.cuda.synchronize()
            best[i] = min(best[i], 1e3 * (time.perf_counter() - t0))
    return best


def test_nearest_point_alone_or_with_its_covariance(lk):
    """The same search but for the list that the covariances are taken from:
    without them the bound is the nearest distance.  (Queries that take some
    thousand probes each: the covariance of one point is some 2 % of them.)"""
    lkc, ctx = lk
    p = workloads.random_cloud(10000, 5, scale=100.0)
    q = dev(p[np.random.default_rng(1).integers(0, len(p), 40000)] + np.float32(8.0))
    t = lkc.lkc_build_target(ctx, dev(p), 1.0)
    alone, cov = _ms(lambda: lkc.lkc_knn_query(ctx, t, q, 1, INF, cfg=WAVE),
                     lambda: lkc.lkc_knn_cov(ctx, t, q, 1, INF, 1e-3, cfg=WAVE))
    assert cov < 1.06 * alone, (cov, alone)
    t.free()


@pytest.mark.parametrize("k", [1, 2, 5, 20, 56, 57, 64])
def test_rings_of_sparse_clouds(lk, k):
    lkc, ctx = lk
    p = workloads.random_cloud(20000, 5, scale=60.0)
    p[100:200] = p[:100]                       # equal distances
    p[5000:5400] = np.round(p[5000:5400])      # a lattice's
    near = p[np.random.default_rng(2).integers(0, len(p), 150)]
    q = np.concatenate([near + np.float32(0.3), near[:60] + np.float32(8.0),
                        near[:40] + np.float32(300.0), p[5000:5050], p[:50]])
    t = lkc.lkc_build_target(ctx, dev(p), 1.0)
    for radius in (INF, 9.0):
        a = {n: v.cpu().numpy() for n, v in
             lkc.lkc_knn_cov(ctx, t, dev(q), k, radius, 1e-3, cfg=WAVE).items()}
        parity.check_knn(p, q, k, radius, a["idx"], a["d2"], a["count"])
    t.free()
