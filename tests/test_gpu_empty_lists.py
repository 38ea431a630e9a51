"""Covariances of neighbour lists that are empty: workgroups of 64 lists with
none, one or all of them empty, and what a call of nothing but such lists costs."""
import time

import numpy as np
import pytest

from paper_2308_07173_amd import workloads
from tests import parity

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


@pytest.mark.parametrize("k", [3, 20, 64])
@pytest.mark.parametrize("kind,sigma", [("none", 0.0), ("gaussian", 0.3)])
@pytest.mark.parametrize("origin", [True, False])
def test_blocks_with_and_without_entries(lk, k, kind, sigma, origin):
    lkc, ctx = lk
    rng = np.random.default_rng(k)
    p = workloads.random_cloud(500, 1)
    q, m = workloads.random_cloud(64 * 6 + 5, 2), 64 * 6 + 5
    idx = rng.integers(0, 500, (m, k)).astype(np.int32)
    cnt = np.full(m, k, np.int32)
    cnt[64:128] = 0                 # a whole workgroup
    cnt[128:192] = 0
    cnt[150] = k                    # all but one
    cnt[200] = 0                    # one
    idx[256:320, 0] = -1            # empty by their first entry
    cnt[-5:] = -3
    t = lkc.lkc_build_target(ctx, torch.from_numpy(p).cuda(), 1.0)
    d = [torch.from_numpy(a).cuda() for a in (idx, cnt, q)]
    o = lkc.lkc_covariances_weighted(ctx, t, d[0], d[1], kind, sigma,
                                     queries=d[2] if origin else None, plane_eps=1e-3)
    o = {key: v.cpu().numpy() for key, v in o.items()}
    n = np.where(idx[:, 0] < 0, 0, np.maximum(cnt, 0))
    assert np.array_equal(o["valid"], n >= 3)
    none = n == 0
    assert (o["mean"][none] == 0).all() and (o["cov"][none] == 0).all()
    assert (o["reg"][none] == np.eye(3, dtype=np.float32)).all()
    keep = np.flatnonzero(~none)
    # the other lists: as in a call without the empty ones
    only = [torch.from_numpy(np.ascontiguousarray(a[keep])).cuda() for a in (idx, cnt, q)]
    ref = lkc.lkc_covariances_weighted(ctx, t, only[0], only[1], kind, sigma,
                                       queries=only[2] if origin else None, plane_eps=1e-3)
    for key, v in ref.items():
        assert np.array_equal(o[key][keep], v.cpu().numpy()), key
    if kind != "none":
        parity.check_cov_weighted(p, idx[keep], n[keep].astype(np.int32), o["mean"][keep],
                                  o["cov"][keep], o["reg"][keep], o["valid"][keep], kind, sigma,
                                  queries=q[keep] if origin else None)
    t.free()


def test_empty_lists_are_not_loaded(lk):
    """A million lists of 64 of which none has an entry: 28 us against 183 of
    the same lists full (with the entries loaded all the same, 100)."""
    lkc, ctx = lk
    p = torch.from_numpy(workloads.random_cloud(100000, 1, scale=50.0)).cuda()
    t = lkc.lkc_build_target(ctx, p, 1.0)
    m = 1_000_000
    idx = ((torch.arange(m, device="cuda")[:, None] + torch.arange(64, device="cuda")) % 100000).int()
    idx = idx.contiguous()
    out = {}

    def ms(cnt):
        best = 1e9
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(4):
                out.update(lkc.lkc_covariances(ctx, t, idx, cnt, out=out or None))
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        return best

    full = ms(torch.full((m,), 64, dtype=torch.int32, device="cuda"))
    none = ms(torch.zeros(m, dtype=torch.int32, device="cuda"))
    assert none < 0.35 * full, (none, full)
    t.free()
