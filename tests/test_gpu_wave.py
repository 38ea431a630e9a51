"""The wavefront-per-query search where its candidate list can go wrong: more
equal distances than the list holds, cells dense enough to be read through
their 16-point runs, lists shorter than k, the step from the wavefront to the
group search, and rebuilds that left the target empty.

Tie clouds lie on an integer lattice, where every float32 d2 is exact: the
lists must equal the oracle's.  Elsewhere the rules of ``tests/parity.py``
hold, and the group search must give the same bits.
"""
import math

import numpy as np
import pytest

from oracle import oracle
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


def host(o):
    return {k: v.cpu().numpy() for k, v in o.items()}


@pytest.mark.parametrize("k", [1, 5, 20, 33, 60, 61, 64])
@pytest.mark.parametrize("radius", [1.0, 2.0, INF])
def test_more_equal_distances_than_the_list_holds(lk, k, radius):
    lkc, ctx = lk
    # 300 copies of each of 9 lattice points: 300, 1200, ... equal distances
    base = workloads.lattice_nd((3, 3, 1), a=1.0)
    rng = np.random.default_rng(3)
    p = base[rng.permutation(np.repeat(np.arange(9), 300))]
    q = np.concatenate([base, base + np.float32(0.5)])
    t = lkc.lkc_build_target(ctx, dev(p), 2.0)
    idx, d2, cnt = (x.cpu().numpy() for x in lkc.lkc_knn_query(ctx, t, dev(q), k, radius, cfg=WAVE))
    o_idx, o_d2, o_cnt = oracle.knn(p, q, k, radius)
    assert np.array_equal(cnt, o_cnt)
    assert np.array_equal(idx, o_idx)
    assert np.array_equal(d2.astype(np.float64), o_d2)
    s = host(lkc.lkc_knn_cov_self(ctx, t, k, radius, 1e-3, cfg=WAVE))
    s_idx, _, s_cnt = oracle.knn(p, p[:200], k, radius)
    assert np.array_equal(s["count"][:200], s_cnt)
    assert np.array_equal(s["idx"][:200], s_idx)
    t.free()


@pytest.mark.parametrize("k", [1, 16, 20, 64])
@pytest.mark.parametrize("n", [1, 15, 63, 64, 65, 257, 6000])
def test_dense_cells(lk, n, k):
    """All points in one cell (at 257 and above through its runs)."""
    lkc, ctx = lk
    p = workloads.random_cloud(n, 11, scale=0.49, offset=(0.5, 0.5, 0.5))
    q = workloads.random_cloud(203, 12, scale=1.5, offset=(0.5, 0.5, 0.5))
    t = lkc.lkc_build_target(ctx, dev(p), 1.0)
    for radius in (0.3, INF):
        g = host(lkc.lkc_knn_cov(ctx, t, dev(q), k, radius, 1e-3, cfg=WAVE))
        parity.check_knn(p, q, k, radius, g["idx"], g["d2"], g["count"])
        s = host(lkc.lkc_knn_cov_self(ctx, t, k, radius, 1e-3, cfg=WAVE))
        parity.check_knn(p, p, k, radius, s["idx"], s["d2"], s["count"],
                         rows=np.arange(0, n, max(1, n // 64)))
    t.free()


@pytest.mark.parametrize("k", [5, 20, 32, 33])
@pytest.mark.parametrize("kernel", ["none", "laplacian"])
def test_wavefront_and_group_search_agree(lk, k, kernel):
    """A scan (dense near the sensor, sparse rings far out) against itself and
    another: more rows than a wavefront keeps for their covariances at a time."""
    lkc, ctx = lk
    p = workloads.single_scan(seed=21)
    q = np.concatenate([workloads.single_scan(seed=22)[:7001],
                        np.array([[np.nan, 0, 0], [900, 900, 900]], np.float32)])
    t = lkc.lkc_build_target(ctx, dev(p), 1.0)
    for a, b in (({}, WAVE), (dict(algorithm=1), WAVE)):
        x = host(lkc.lkc_knn_cov_weighted(ctx, t, dev(q), k, kernel, 0.2, 2.0, 1e-3, cfg=a))
        y = host(lkc.lkc_knn_cov_weighted(ctx, t, dev(q), k, kernel, 0.2, 2.0, 1e-3, cfg=b))
        for key in x:
            assert np.array_equal(x[key], y[key]), key
    x = host(lkc.lkc_knn_cov_self(ctx, t, k, 2.0, 1e-3, cfg=dict(algorithm=1)))
    y = host(lkc.lkc_knn_cov_self(ctx, t, k, 2.0, 1e-3, cfg=WAVE))
    for key in x:
        assert np.array_equal(x[key], y[key]), key
    t.free()


@pytest.mark.parametrize("n", [98304, 98305])
def test_either_side_of_the_step_to_the_group_search(lk, n):
    lkc, ctx = lk
    p = workloads.single_scan(seed=23)
    q = np.tile(workloads.single_scan(seed=24), (2, 1))[:n]
    t = lkc.lkc_build_target(ctx, dev(p), 1.0)
    x = host(lkc.lkc_knn_cov(ctx, t, dev(q), 20, 2.0, 1e-3))
    assert (ctx.search_stats()["fallback_queries"] == n) == (n <= 98304)
    y = host(lkc.lkc_knn_cov(ctx, t, dev(q), 20, 2.0, 1e-3,
                             cfg=dict(algorithm=1 if n <= 98304 else 2)))
    for key in x:
        assert np.array_equal(x[key], y[key]), key
    t.free()


def test_self_search_of_a_target_a_failed_rebuild_emptied(lk):
    lkc, ctx = lk
    p = workloads.plane_wall(1500, seed=2)
    t = lkc.lkc_build_target(ctx, dev(p), 1.0)
    bad = p.copy()
    bad[700] = np.nan
    t.rebuild(dev(bad), sync=False)
    out = lkc.lkc_knn_cov_self(ctx, t, 10, INF, 1e-3,
                               out=dict(idx=torch.full((1500, 10), 7, dtype=torch.int32).cuda(),
                                        d2=torch.zeros(1500, 10).cuda(),
                                        count=torch.full((1500,), 7, dtype=torch.int32).cuda(),
                                        mean=torch.ones(1500, 3).cuda(),
                                        cov=torch.ones(1500, 3, 3).cuda(),
                                        reg=torch.zeros(1500, 3, 3).cuda(),
                                        valid=torch.ones(1500, dtype=torch.uint8).cuda()))
    assert t.status() != lkc.LKC_OK
    o = host(out)
    assert (o["count"] == 0).all() and (o["idx"] == -1).all() and not o["valid"].any()
    assert np.isinf(o["d2"]).all() and (o["mean"] == 0).all() and (o["cov"] == 0).all()
    assert (o["reg"] == np.eye(3, dtype=np.float32)).all()
    t.free()
