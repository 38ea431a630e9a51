"""Targets small enough to be sorted by counting, around the sizes where its
workgroups end and where the radix sort takes over: many equal keys, one cell,
cells of one point, first builds and both kinds of rebuild."""
import math

import numpy as np
import pytest

from paper_2308_07173_amd import workloads
from tests import parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def cloud(kind, n):
    rng = np.random.default_rng(n)
    if kind == "copies":      # 9 points, n / 9 copies of each: equal keys
        base = workloads.lattice_nd((3, 3, 1), a=1.0)
        return base[rng.integers(0, 9, n)]
    if kind == "one cell":
        return workloads.random_cloud(n, 4, scale=0.2, offset=(0.5, 0.5, 0.5))
    return workloads.random_cloud(n, 5, scale=40.0)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1024, 1025, 2049, 8191, 8192, 8193])
@pytest.mark.parametrize("kind", ["copies", "one cell", "sparse"])
def test_layout_by_counting(n, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_07173_amd import lkc
    ctx = lkc.Context()
    p = cloud(kind, n).astype(np.float32)
    d = torch.from_numpy(p).cuda()
    t = lkc.lkc_build_target(ctx, d, 1.0)
    cells = np.unique(np.floor(p).astype(np.int64), axis=0).shape[0]
    layouts = []
    for sync in (None, True, False):
        if sync is not None:
            t.rebuild(d, sync=sync)
        pts, start, keys = (x.cpu().numpy() for x in t.arrays())
        assert len(keys) == cells and len(np.unique(keys)) == cells
        assert start[0] == 0 and start[-1] == n and np.all(np.diff(start.astype(np.int64)) > 0)
        order = np.ascontiguousarray(pts[:n, 3]).view(np.int32)
        assert np.array_equal(np.sort(order), np.arange(n))
        assert np.array_equal(pts[:n, :3], p[order])
        # the points of a cell together; copies in their original order
        cell_of = np.floor(p[order]).astype(np.int64)
        same = np.all(cell_of[1:] == cell_of[:-1], axis=1)
        assert int((~same).sum()) + 1 == cells
        eq = np.all(p[order[1:]] == p[order[:-1]], axis=1)
        assert np.all(order[1:][eq] > order[:-1][eq])
        layouts.append((order, start, keys))
    for o in layouts[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(layouts[0], o))
    idx, d2, cnt = (x.cpu().numpy() for x in lkc.lkc_knn_query(ctx, t, d[:300], 8, math.inf))
    parity.check_knn(p, p[:300], 8, math.inf, idx, d2, cnt)
    t.free()
    ctx.close()
