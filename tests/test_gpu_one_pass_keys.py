"""Targets of few points whose key is one radix pass: they are sorted by
counting up to 4,096 points only, where others are up to 8,192."""
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


def one_cell(n):
    return torch.from_numpy(workloads.random_cloud(n, 4, scale=0.3, offset=(5.5, 5.5, 5.5))).cuda()


@pytest.mark.parametrize("n", [4095, 4096, 4097, 8192])
def test_layout_either_side(lk, n):
    """Points in the Morton order of their quarter-metre sub-cells, those of one
    sub-cell as they came; by all three builds."""
    lkc, ctx = lk
    d = one_cell(n)
    p = d.cpu().numpy()
    t = lkc.lkc_build_target(ctx, d, 1.0)
    assert t.info()["sort_passes"] == 1
    sub = np.floor((p - np.float32(5.0)) * np.float32(4.0)).astype(np.int64)
    key = np.zeros(n, np.int64)
    for bit in range(2):
        for a in range(3):
            key |= ((sub[:, a] >> bit) & 1) << (3 * bit + a)
    want = np.argsort(key, kind="stable")
    for sync in (None, True, False):
        if sync is not None:
            t.rebuild(d, sync=sync)
        pts, start, _ = (x.cpu().numpy() for x in t.arrays())
        assert start.tolist() == [0, n]
        assert np.array_equal(np.ascontiguousarray(pts[:n, 3]).view(np.int32), want)
    # a cloud that needs more passes, rebuilt from those of one
    q = torch.from_numpy(workloads.random_cloud(n, 5, scale=30.0)).cuda()
    t.rebuild(q)
    ref = lkc.lkc_build_target(ctx, q, 1.0)
    for a, b in zip(t.arrays(), ref.arrays()):
        assert torch.equal(a, b)
    t.free()
    ref.free()


def test_counting_stops_where_a_pass_costs_less(lk):
    """8,192 points of one cell, rebuilt: 32 us by counting, 25 by a pass."""
    lkc, ctx = lk

    def ms(n):
        d = one_cell(n)
        t = lkc.lkc_build_target(ctx, d, 1.0)
        best = math.inf
        for _ in range(20):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(50):
                t.rebuild(d, sync=False)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        t.free()
        return best

    few, more = ms(8192), ms(8193)
    assert few < 1.12 * more, (few, more)
