"""Searches of more than 56 neighbours, whose candidate lists keep 128 entries:
around that step, with more equal distances than the list holds, cells of a
few and of thousands of points, plain and weighted.  Lattices must equal the
oracle, the rest follows the rules of ``tests/parity.py``."""
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


@pytest.mark.parametrize("k", [56, 57, 60, 63, 64])
@pytest.mark.parametrize("copies", [63, 64, 65, 127, 128, 129, 193, 700])
def test_equal_distances(lk, k, copies):
    lkc, ctx = lk
    base = workloads.lattice_nd((3, 2, 1), a=1.0)
    rng = np.random.default_rng(copies)
    p = base[rng.permutation(np.repeat(np.arange(6), copies))]
    p = np.concatenate([p, workloads.random_cloud(4097, 1, scale=20.0, offset=(500.0, 0, 0))])
    p = p.astype(np.float32)
    q = np.concatenate([base, base + np.float32(0.5)])
    t = lkc.lkc_build_target(ctx, dev(p), 2.0)
    for radius in (0.5, 1.0, 9.0):
        idx, d2, cnt = (x.cpu().numpy() for x in lkc.lkc_knn_query(ctx, t, dev(q), k, radius))
        o_idx, o_d2, o_cnt = oracle.knn(p, q, k, radius)
        assert np.array_equal(cnt, o_cnt)
        assert np.array_equal(idx, o_idx)
        assert np.array_equal(d2.astype(np.float64), o_d2)
    s = host(lkc.lkc_knn_cov_self(ctx, t, k, 3.0, 1e-3))
    s_idx, _, s_cnt = oracle.knn(p, p[:150], k, 3.0)
    assert np.array_equal(s["count"][:150], s_cnt)
    assert np.array_equal(s["idx"][:150], s_idx)
    t.free()


@pytest.mark.parametrize("k", [57, 61, 64])
@pytest.mark.parametrize("kind,sigma", [("none", 0.0), ("laplacian", 0.2), ("gaussian", 0.3)])
def test_rows_and_covariances(lk, k, kind, sigma):
    """More rows than a wavefront keeps, lists shorter than k among them; the
    fused call equals the two calls."""
    lkc, ctx = lk
    p = workloads.single_scan(seed=31)[:30000]
    q = np.concatenate([workloads.single_scan(seed=32)[:9001], np.full((1, 3), 800.0)])
    q = q.astype(np.float32)
    t = lkc.lkc_build_target(ctx, dev(p), 1.0)
    qd = dev(q)
    f = lkc.lkc_knn_cov_weighted(ctx, t, qd, k, kind, sigma, 1.0, 1e-3)
    idx, d2, cnt = lkc.lkc_knn_query(ctx, t, qd, k, 1.0)
    c = lkc.lkc_covariances_weighted(ctx, t, idx, cnt, kind, sigma, queries=qd, plane_eps=1e-3)
    assert torch.equal(idx, f["idx"]) and torch.equal(d2, f["d2"]) and torch.equal(cnt, f["count"])
    for key in ("mean", "cov", "reg", "valid"):
        assert torch.equal(c[key], f[key]), key
    n = cnt.cpu().numpy()
    assert (n < k).any() and (n == k).any()
    rows = np.arange(0, len(q), 97)
    parity.check_knn(p, q, k, 1.0, idx.cpu().numpy(), d2.cpu().numpy(), n, rows=rows)
    t.free()


def test_sixty_four_neighbours_cost_about_as_much_as_fifty_six(lk):
    """In one cell of 10,000 points the candidates come in no useful order and
    the list is cut over and over (with 64 entries, five times the time)."""
    lkc, ctx = lk
    t = lkc.lkc_build_target(ctx, dev(workloads.random_cloud(10000, 1, scale=0.45)), 10.0)

    def ms(k):
        out = lkc.lkc_knn_cov_self(ctx, t, k, 1.0, 1e-3)
        best = INF
        for _ in range(5):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(3):
                lkc.lkc_knn_cov_self(ctx, t, k, 1.0, 1e-3, out=out)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        return best

    at56, at64 = ms(56), ms(64)
    assert at64 < 2.0 * at56, (at56, at64)
    t.free()
