"""The group search asked for by name, where searches of this size take the
wavefront search by themselves: targets that it streams whole, equal
distances, empty and non-finite queries, weights, batches over several
targets.  What it hands on is counted, so that it cannot be the other search
that answers.  Lattices must equal the oracle, the rest follows the rules of
``tests/parity.py``; the wavefront search gives the same bits."""
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
SHAPES = [dict(algorithm=1), dict(algorithm=1, group_split=1), dict(algorithm=1, group_split=4),
          dict(algorithm=1, persistent=2), dict(algorithm=1, group_reach=3, waves_per_block=4)]


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


def grouped(ctx, q, share=0.9):
    """The groups answered at least a part of the queries themselves."""
    s = ctx.search_stats()
    assert s["queries"] == q and s["fallback_queries"] <= share * q, s


def same(a, b):
    for key in a:
        assert np.array_equal(a[key], b[key]), key


@pytest.mark.parametrize("cfg", SHAPES)
@pytest.mark.parametrize("n", [4096, 4097])
def test_whole_target_boundary(lk, n, cfg):
    lkc, ctx = lk
    p = workloads.plane_wall(n, seed=31)
    q = np.concatenate([p[:2500] + np.float32(0.03), workloads.random_cloud(500, 32, scale=12.0)])
    t = lkc.lkc_build_target(ctx, dev(p), 1.0)
    for radius in (1.0, INF):
        a = host(lkc.lkc_knn_cov_self(ctx, t, 12, radius, 1e-3, cfg=cfg))
        grouped(ctx, n)
        b = host(lkc.lkc_knn_cov(ctx, t, dev(q), 12, radius, 1e-3, cfg=cfg))
        grouped(ctx, len(q))
        same(a, host(lkc.lkc_knn_cov_self(ctx, t, 12, radius, 1e-3, cfg=WAVE)))
        same(b, host(lkc.lkc_knn_cov(ctx, t, dev(q), 12, radius, 1e-3, cfg=WAVE)))
        for qs, o in ((p, a), (q, b)):
            rows = np.arange(qs.shape[0])[::7]
            parity.check_knn(p, qs, 12, radius, o["idx"], o["d2"], o["count"], rows=rows)
            parity.check_cov(p, o["idx"], o["count"], o["mean"], o["cov"], o["reg"],
                             o["valid"], rows=rows, search=(qs, 12, radius))
    t.free()


@pytest.mark.parametrize("k", [1, 4, 7, 20, 32])
@pytest.mark.parametrize("shape,cell", [((90, 80), 2.0), ((20, 18, 16), 1.0), ((64, 70), 0.75)])
def test_lattices(lk, shape, cell, k):
    """Every distance many times over, ties decided by the index."""
    lkc, ctx = lk
    p = workloads.lattice_nd(shape)
    p = p[np.random.default_rng(1).permutation(len(p))]
    q = np.concatenate([p[:700], p[:300] + np.float32(0.5)])
    t = lkc.lkc_build_target(ctx, dev(p), cell)
    for radius in (1.0, 3.0):
        idx, d2, cnt = (x.cpu().numpy() for x in
                        lkc.lkc_knn_query(ctx, t, dev(q), k, radius, cfg=SHAPES[0]))
        assert ctx.search_stats()["queries"] == len(q)
        o_idx, o_d2, o_cnt = oracle.knn(p, q, k, radius)
        assert np.array_equal(cnt, o_cnt) and np.array_equal(idx, o_idx)
        assert np.array_equal(d2.astype(np.float64), o_d2)
        s = host(lkc.lkc_knn_cov_self(ctx, t, k, radius, 1e-3, cfg=SHAPES[0]))
        same(s, host(lkc.lkc_knn_cov_self(ctx, t, k, radius, 1e-3, cfg=WAVE)))
        s_idx, _, _ = oracle.knn(p, p[:300], k, radius)
        assert np.array_equal(s["idx"][:300], s_idx)
    t.free()


@pytest.mark.parametrize("cfg", SHAPES)
@pytest.mark.parametrize("n", [0, 3, 700, 9000])
def test_empty_short_and_non_finite(lk, n, cfg):
    lkc, ctx = lk
    p = workloads.random_cloud(n, 3, scale=6.0)
    q = workloads.random_cloud(900, 4, scale=6.0)
    q[5] = np.nan
    q[64:128] = np.inf           # a whole group's worth
    q[700, 2] = -np.inf
    q[800:] += 500.0             # nothing within the radius
    t = lkc.lkc_build_target(ctx, dev(p) if n else torch.zeros(0, 3, device="cuda"), 1.0)
    o = host(lkc.lkc_knn_cov(ctx, t, dev(q), 20, 2.0, 1e-3, cfg=cfg))
    grouped(ctx, 900)
    same(o, host(lkc.lkc_knn_cov(ctx, t, dev(q), 20, 2.0, 1e-3, cfg=WAVE)))
    none = ~np.isfinite(q).all(axis=1)
    none[800:] = True
    if n == 0:
        none[:] = True
    assert (o["count"][none] == 0).all() and (o["idx"][none] == -1).all()
    assert np.isinf(o["d2"][none]).all() and not o["valid"][none].any()
    if n:
        rows = np.flatnonzero(~none)[::5]
        parity.check_knn(p, q, 20, 2.0, o["idx"], o["d2"], o["count"], rows=rows)
    t.free()


@pytest.mark.parametrize("kind,sigma", [("laplacian", 0.2), ("gaussian", 0.3), ("rbf", 4.0)])
@pytest.mark.parametrize("k", [5, 8, 20, 32])
def test_weights(lk, kind, sigma, k):
    lkc, ctx = lk
    p = workloads.single_scan(seed=41)[:40000]
    q = np.concatenate([workloads.single_scan(seed=41)[40000:47000], p[:2001]])
    t = lkc.lkc_build_target(ctx, dev(p), 1.0)
    qd = dev(q)
    g = lkc.lkc_knn_cov_weighted(ctx, t, qd, k, kind, sigma, 2.0, 1e-3, cfg=SHAPES[0])
    grouped(ctx, len(q))
    w = lkc.lkc_knn_cov_weighted(ctx, t, qd, k, kind, sigma, 2.0, 1e-3, cfg=WAVE)
    c = lkc.lkc_covariances_weighted(ctx, t, g["idx"], g["count"], kind, sigma, queries=qd,
                                     plane_eps=1e-3)
    same(host(g), host(w))
    for key in ("mean", "cov", "reg", "valid"):
        assert torch.equal(g[key], c[key]), key
    o = host(g)
    rows = np.arange(0, len(q), 61)
    parity.check_knn(p, q, k, 2.0, o["idx"], o["d2"], o["count"], rows=rows)
    # (the lists as the search gave them, checked above: the oracle weighs the same)
    parity.check_cov_weighted(p, o["idx"], o["count"], o["mean"], o["cov"], o["reg"], o["valid"],
                              kind, sigma, queries=q, rows=rows)
    t.free()


@pytest.mark.parametrize("cfg", SHAPES + [WAVE])
@pytest.mark.parametrize("k", [5, 20])
def test_batches_over_several_targets(lk, cfg, k):
    """Uneven scans against a small, a large, an empty and a flat target: each
    scan's rows are those of the scan alone, in either search."""
    lkc, ctx = lk
    clouds = [workloads.plane_wall(3000, seed=1), workloads.single_scan(seed=2),
              np.zeros((0, 3), np.float32),
              workloads.random_cloud(9000, 3) * np.array([60, 40, 0.1], np.float32)]
    targets = [lkc.lkc_build_target(ctx, dev(c) if len(c) else torch.zeros(0, 3, device="cuda"), cell)
               for c, cell in zip(clouds, (0.5, 1.0, 1.0, 2.0))]
    rng = np.random.default_rng(5)
    scans, parts, at = [], [], 0
    for i, n in enumerate([900, 4000, 65, 2500, 63, 1, 3000, 64, 0, 1800]):
        w = i % 4
        src = clouds[w] if len(clouds[w]) else clouds[0]
        parts.append(src[rng.integers(0, len(src), n)] + rng.normal(0, 0.05, (n, 3)).astype(np.float32))
        scans.append((at, n, w))
        at += n
    q = np.concatenate(parts).astype(np.float32)
    ts = lkc.TargetSet(ctx, targets, 16)
    ts.stage(scans)
    got = host(lkc.lkc_knn_cov_batched(ctx, ts, dev(q), k, 2.0, 1e-3, cfg=cfg))
    if cfg is not WAVE:
        grouped(ctx, at)
    for (o, n, w), part in zip(scans, parts):
        for other in (SHAPES[0], WAVE):
            alone = host(lkc.lkc_knn_cov(ctx, targets[w], dev(q[o:o + n]), k, 2.0, 1e-3, cfg=other))
            for key in alone:
                assert np.array_equal(got[key][o:o + n], alone[key]), (key, w)
    ts.free()
    for t in targets:
        t.free()
