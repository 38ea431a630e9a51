"""Queries that cost far more than others, next to each other in the order in
which the wavefront search takes them: they must not fall to one part of the
device.  And numbers of queries at which its shares of them change."""
import math
import time

import numpy as np
import pytest

from paper_2308_07173_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

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


@pytest.mark.parametrize("q", [1, 7, 8, 31, 32, 33, 127, 128, 255, 256, 257, 2047, 2049, 24575,
                               24577, 65535, 131073])
def test_every_query_once(lk, q):
    lkc, ctx = lk
    p = workloads.plane_wall(6000, seed=3)
    t = lkc.lkc_build_target(ctx, dev(p), 1.0)
    qs = dev(np.tile(p, (22, 1))[:q] + np.float32(0.01))
    out = dict(idx=torch.full((q, 4), -7, dtype=torch.int32, device="cuda"),
               d2=torch.full((q, 4), -7.0, device="cuda"),
               count=torch.full((q,), -7, dtype=torch.int32, device="cuda"),
               mean=torch.zeros(q, 3, device="cuda"), cov=torch.zeros(q, 3, 3, device="cuda"),
               reg=torch.zeros(q, 3, 3, device="cuda"),
               valid=torch.full((q,), 7, dtype=torch.uint8, device="cuda"))
    lkc.lkc_knn_cov(ctx, t, qs, 4, math.inf, 1e-3, out=out, cfg=WAVE)
    ref = lkc.lkc_knn_cov(ctx, t, qs, 4, math.inf, 1e-3, cfg=dict(algorithm=1))
    for key in ref:
        assert torch.equal(out[key], ref[key]), key
    t.free()


def test_order_of_costly_queries(lk):
    """An eighth of the queries in a sparse part, after the others or among them."""
    lkc, ctx = lk
    dense = workloads.random_cloud(20000, 1, scale=5.0)
    sparse = workloads.random_cloud(4000, 2, scale=100.0, offset=(200.0, 0, 0))
    t = lkc.lkc_build_target(ctx, dev(np.concatenate([dense, sparse])), 1.0)
    q = np.concatenate([workloads.random_cloud(57344, 3, scale=5.0),
                        workloads.random_cloud(8192, 4, scale=100.0, offset=(200.0, 0, 0))])
    at = np.random.default_rng(0).permutation(len(q))
    after, among = dev(q), dev(q[at])

    def ms(x):
        out = lkc.lkc_knn_cov(ctx, t, x, 10, math.inf, 1e-3, cfg=WAVE)
        best = math.inf
        for _ in range(4):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            lkc.lkc_knn_cov(ctx, t, x, 10, math.inf, 1e-3, out=out, cfg=WAVE)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        return best, out

    (t_after, a), (t_among, b) = ms(after), ms(among)
    for key in a:
        assert torch.equal(a[key][torch.from_numpy(at).cuda()], b[key]), key
    assert t_after < 2.0 * t_among, (t_after, t_among)
    t.free()
