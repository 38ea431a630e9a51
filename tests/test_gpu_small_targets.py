"""Targets of few points, which the wavefront search takes as a whole: at the
edges of its runs and of the size up to which it does, however far apart the
points and the queries lie, and in batches beside large targets.

Lattices, whose float32 d2 are exact, must equal the oracle; elsewhere the
rules of ``tests/parity.py`` hold, and the group search gives the same bits.
"""
import math
import time

import numpy as np
import pytest

from oracle import oracle
from paper_2308_07173_amd import workloads
from tests import parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

INF = math.inf
WAVE, GROUP = dict(algorithm=2), dict(algorithm=1)


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


@pytest.mark.parametrize("k", [1, 16, 17, 32, 64])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 255, 256, 257, 1023, 1025, 4095, 4096, 4097])
def test_sizes(lk, n, k):
    lkc, ctx = lk
    p = workloads.random_cloud(n, n, scale=30.0)
    q = np.concatenate([workloads.random_cloud(130, 1, scale=30.0),
                        workloads.random_cloud(40, 2, scale=3.0, offset=(400.0, -90.0, 7.0)),
                        p[:7], np.array([[np.nan, 0, 0]], np.float32)])
    t = lkc.lkc_build_target(ctx, dev(p), 1.0)
    for radius in (INF, 12.0, 0.5):
        a = host(lkc.lkc_knn_cov(ctx, t, dev(q), k, radius, 1e-3, cfg=WAVE))
        parity.check_knn(p, q, k, radius, a["idx"], a["d2"], a["count"])
        s = host(lkc.lkc_knn_cov_self(ctx, t, k, radius, 1e-3, cfg=WAVE))
        rows = np.arange(0, n, max(1, n // 64))
        parity.check_knn(p, p, k, radius, s["idx"], s["d2"], s["count"], rows=rows)
        if k <= 32:
            b = host(lkc.lkc_knn_cov(ctx, t, dev(q), k, radius, 1e-3, cfg=GROUP))
            r = host(lkc.lkc_knn_cov_self(ctx, t, k, radius, 1e-3, cfg=GROUP))
            for key in a:
                assert np.array_equal(a[key], b[key]), key
                assert np.array_equal(s[key], r[key]), key
    t.free()


@pytest.mark.parametrize("k", [1, 5, 20, 33, 64])
@pytest.mark.parametrize("others", [0, 4097])
def test_ties_in_either_search(lk, k, others):
    """Many equal distances, in a target taken as a whole and (beside points
    out of reach) in one whose cells are searched."""
    lkc, ctx = lk
    base = workloads.lattice_nd((3, 3, 1), a=1.0)
    rng = np.random.default_rng(3)
    p = base[rng.permutation(np.repeat(np.arange(9), 300))]
    far = workloads.random_cloud(others, 5, scale=40.0, offset=(900.0, 900.0, 0.0))
    p = np.concatenate([p, far]).astype(np.float32)
    q = np.concatenate([base, base + np.float32(0.5)])
    t = lkc.lkc_build_target(ctx, dev(p), 2.0)
    for radius in (1.0, 2.0, 5.0):
        idx, d2, cnt = (x.cpu().numpy() for x in
                        lkc.lkc_knn_query(ctx, t, dev(q), k, radius, cfg=WAVE))
        o_idx, o_d2, o_cnt = oracle.knn(p, q, k, radius)
        assert np.array_equal(cnt, o_cnt)
        assert np.array_equal(idx, o_idx)
        assert np.array_equal(d2.astype(np.float64), o_d2)
        s = host(lkc.lkc_knn_cov_self(ctx, t, k, radius, 1e-3, cfg=WAVE))
        s_idx, _, s_cnt = oracle.knn(p, p[:200], k, radius)
        assert np.array_equal(s["count"][:200], s_cnt)
        assert np.array_equal(s["idx"][:200], s_idx)
    t.free()


@pytest.mark.parametrize("n", [1, 63, 257, 2048])
def test_one_dense_cell_beside_far_points(lk, n):
    """Dense cells of a target whose cells are searched (its other points out
    of reach), read whole and through their runs."""
    lkc, ctx = lk
    p = np.concatenate([workloads.random_cloud(n, 11, scale=0.49, offset=(0.5, 0.5, 0.5)),
                        workloads.random_cloud(4097, 12, scale=30.0, offset=(300.0, 0.0, 0.0))])
    q = workloads.random_cloud(203, 13, scale=1.5, offset=(0.5, 0.5, 0.5))
    t = lkc.lkc_build_target(ctx, dev(p), 1.0)
    for k in (1, 20, 64):
        for radius in (0.3, 3.0):
            g = host(lkc.lkc_knn_cov(ctx, t, dev(q), k, radius, 1e-3, cfg=WAVE))
            parity.check_knn(p, q, k, radius, g["idx"], g["d2"], g["count"])
    t.free()


@pytest.mark.parametrize("algorithm", [0, 1, 2])
@pytest.mark.parametrize("radius", [INF, 2.0, 9.0])
def test_batches_over_small_and_large_targets(lk, algorithm, radius):
    lkc, ctx = lk
    clouds = [workloads.random_cloud(300, 1, scale=60.0), workloads.single_scan(seed=4)[:20000],
              workloads.random_cloud(4096, 2, scale=20.0)]
    targets = [lkc.lkc_build_target(ctx, dev(c), 1.0) for c in clouds]
    scans = [workloads.random_cloud(m, 10 + i, scale=40.0) for i, m in enumerate((500, 700, 901, 333))]
    which = [0, 1, 2, 0]
    for use in ([0, 1, 2], [0, 2]):
        ts = lkc.TargetSet(ctx, [targets[i] for i in use], 8)
        table, at, picked = [], 0, []
        for s, w in zip(scans, which):
            if w in use:
                table.append((at, len(s), use.index(w)))
                at += len(s)
                picked.append((s, w))
        ts.stage(table)
        q = np.concatenate([s for s, _ in picked])
        got = host(lkc.lkc_knn_cov_batched(ctx, ts, dev(q), 10, radius, 1e-3,
                                           cfg=dict(algorithm=algorithm)))
        at = 0
        for s, w in picked:
            one = host(lkc.lkc_knn_cov(ctx, targets[w], dev(s), 10, radius, 1e-3, cfg=WAVE))
            for key in one:
                assert np.array_equal(got[key][at:at + len(s)], one[key]), (key, w)
            at += len(s)
        ts.free()
    for t in targets:
        t.free()


def _ms(fn):
    fn()
    best = INF
    for _ in range(5):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(3):
            fn()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t0)
    return best


@pytest.mark.parametrize("n", [300, 2048, 4096])
def test_sparse_target_without_a_radius_costs_no_more_than_groups(lk, n):
    """Points tens of cells apart: by rings of cells such a search takes 10 to
    40 times the group search, which streams the target whole."""
    lkc, ctx = lk
    p = dev(workloads.random_cloud(n, n, scale=100.0))
    q = dev(workloads.random_cloud(40000, 1, scale=100.0))
    t = lkc.lkc_build_target(ctx, p, 1.0)
    wave = _ms(lambda: lkc.lkc_knn_cov(ctx, t, q, 5, INF, 1e-3))
    group = _ms(lambda: lkc.lkc_knn_cov(ctx, t, q, 5, INF, 1e-3, cfg=GROUP))
    assert wave < 2.0 * group, (wave, group)
    t.free()


@pytest.mark.parametrize("k", [3, 4, 20, 64])
@pytest.mark.parametrize("n", [4097, 10000, 16384, 16385])
def test_sparse_targets_of_more_points(lk, n, k):
    """Either side of the size up to which a sparse target is taken as a whole
    (k >= 4, no radius or a large one)."""
    lkc, ctx = lk
    p = workloads.random_cloud(n, n, scale=100.0)
    q = np.concatenate([workloads.random_cloud(300, 1, scale=100.0), p[:40]])
    t = lkc.lkc_build_target(ctx, dev(p), 1.0)
    for radius in (INF, 25.0, 1.5):
        a = host(lkc.lkc_knn_cov(ctx, t, dev(q), k, radius, 1e-3, cfg=WAVE))
        parity.check_knn(p, q, k, radius, a["idx"], a["d2"], a["count"])
        s = host(lkc.lkc_knn_cov_self(ctx, t, k, radius, 1e-3, cfg=WAVE))
        parity.check_knn(p, p, k, radius, s["idx"], s["d2"], s["count"], rows=np.arange(0, n, 97))
        if k <= 32:
            for key, v in host(lkc.lkc_knn_cov(ctx, t, dev(q), k, radius, 1e-3, cfg=GROUP)).items():
                assert np.array_equal(a[key], v), key
    t.free()


def test_sparse_target_of_ten_thousand_points(lk):
    """By rings 36 times the target of 4,096 points as sparse, which is taken as
    a whole; so 1.4 times."""
    lkc, ctx = lk
    q = dev(workloads.random_cloud(40000, 1, scale=100.0))

    def ms(n):
        t = lkc.lkc_build_target(ctx, dev(workloads.random_cloud(n, n, scale=100.0)), 1.0)
        r = _ms(lambda: lkc.lkc_knn_cov(ctx, t, q, 5, INF, 1e-3))
        t.free()
        return r

    few, more = ms(4096), ms(10000)
    assert more < 5.0 * few, (few, more)
