"""Clustering of clouds for which its passes over the pairs differ: two to 64
points a wavefront, cells long enough to be read by all lanes, half a million
points and more (a lane per point, one pass of joins, wavefronts with few kept
points).  All clouds have labels that are known without a reference."""
import math
import time

import numpy as np
import pytest

from paper_2308_07173_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_07173_amd import lkc
    ctx = lkc.Context()
    yield lkc, ctx
    ctx.close()


def dev(a, dtype=np.float32):
    return torch.from_numpy(np.ascontiguousarray(a, dtype)).cuda()


def labels_of(group, kept):
    """Smallest kept index of every kept point's group, -1 elsewhere."""
    n = len(group)
    first = np.full(int(group.max()) + 1, n)
    np.minimum.at(first, group[kept], np.flatnonzero(kept))
    return np.where(kept, first[group], -1)


def check(lk, p, eps, group, mask=None):
    """group: component of every point if all are kept (a mask may not split one)."""
    lkc, ctx = lk
    kept = np.ones(len(p), bool) if mask is None else mask.astype(bool)
    want = labels_of(group, kept)
    count = len(np.unique(want[kept])) if kept.any() else 0
    md = None if mask is None else dev(mask, np.uint8)
    labels, k = lkc.lkc_euclid_cluster(ctx, dev(p), eps, mask=md)
    assert k == count and np.array_equal(labels.cpu().numpy(), want)
    for _ in range(2):
        o = lkc.lkc_euclid_cluster_async(ctx, dev(p), eps, mask=md)
        assert int(o["status"]) == 0 and int(o["n_clusters"]) == count
        assert np.array_equal(o["labels"].cpu().numpy(), want)


@pytest.mark.parametrize("n", [65536, 65537, 131073, 262145, 524288, 524289, 1100001])
@pytest.mark.parametrize("keep", [None, 0.02, 0.6])
def test_chains(lk, n, keep):
    """A line cut every 50 points, in random order; cut where the mask drops points."""
    rng = np.random.default_rng(n)
    at = rng.permutation(n)                       # position of every point
    mask = None
    gap = at // 50
    if keep is not None:
        on = rng.random(n) < keep                 # by position
        mask = on[at].astype(np.uint8)
        start = np.r_[True, (on[1:] != on[:-1]) | (np.arange(1, n) % 50 == 0)]
        gap = (np.cumsum(start) - 1)[at]
    p = np.zeros((n, 3), np.float32)
    p[:, 0] = (at % 50000) * 0.25 + ((at // 50) % 1000) * 0.75
    p[:, 1] = (at // 50000) * 4.0
    check(lk, p, 0.25, gap, mask)


@pytest.mark.parametrize("copies", [1, 31, 33, 64, 65, 300, 2000])
def test_spots(lk, copies):
    """Many points in a place, beside single ones: long cells among short."""
    rng = np.random.default_rng(copies)
    spots = np.stack(np.meshgrid(np.arange(5), np.arange(4), np.arange(2), indexing="ij"), -1)
    spots = spots.reshape(-1, 3).astype(np.float32) * 0.6
    single = np.stack(np.meshgrid(np.arange(60), np.arange(50), [5.0], indexing="ij"), -1)
    single = single.reshape(-1, 3).astype(np.float32) * 0.6
    p = np.concatenate([np.repeat(spots, copies, axis=0), single])
    group = np.concatenate([np.repeat(np.arange(40), copies), 40 + np.arange(3000)])
    order = rng.permutation(len(p))
    p, group = p[order], group[order]
    check(lk, p, 0.5, group)                                        # every spot by itself
    check(lk, p, 0.7, np.where(group < 40, 0, 1))                   # two sheets
    keep = rng.random(len(p)) < 0.3
    check(lk, p, 0.5, group, keep.astype(np.uint8))


def test_a_volume_of_pairs(lk):
    """Hardly more points than cells, evenly: one pass of joins; kept by half,
    and with a line of the same points beside it, the others."""
    side = 66
    g = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3) * 2.5
    p = np.concatenate([g, g + [0.9, 0, 0]]).astype(np.float32)
    n = len(p)
    assert n > (1 << 19)
    group = np.tile(np.arange(len(g)), 2)
    order = np.random.default_rng(0).permutation(n)
    p, group = p[order], group[order]
    check(lk, p, 1.5, group)
    check(lk, p, 1.5, group, (np.random.default_rng(1).random(n) < 0.5).astype(np.uint8))
    far = np.zeros((20000, 3), np.float32)
    far[:, 0] = np.arange(20000) + 1e4
    far[:, 1] = 1e4
    check(lk, np.concatenate([p, far]), 1.5, np.concatenate([group, np.full(20000, n)]))


@pytest.mark.parametrize("eps,one", [(0.9, False), (1.0, True)])
def test_a_sheet(lk, eps, one):
    g = np.stack(np.meshgrid(np.arange(900), np.arange(700), [0.0], indexing="ij"), -1)
    p = g.reshape(-1, 3).astype(np.float32)
    p = p[np.random.default_rng(2).permutation(len(p))]
    check(lk, p, eps, np.zeros(len(p), np.int64) if one else np.arange(len(p)))


def test_long_cells_cost_no_more_than_short_ones(lk):
    """20,000 points in 20 places against as many apart.  With a lane to a cell
    the first took 1.53 ms, the second 0.13."""
    lkc, ctx = lk

    def ms(p, eps):
        d = dev(p)
        o = lkc.lkc_euclid_cluster_async(ctx, d, eps)
        best = math.inf
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(5):
                lkc.lkc_euclid_cluster_async(ctx, d, eps, out=o)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        return best

    spots = np.repeat(workloads.random_cloud(20, 1, scale=10.0), 1000, axis=0)
    apart = workloads.random_cloud(20000, 2, scale=10.0)
    a, b = ms(spots, 0.5), ms(apart, 0.2)
    assert a < 4.0 * b, (a, b)
