"""Calls so large that a launch with several threads an item would hold 2^32
threads or more, past what a launch may have.  The answers are known without
a reference: a lattice whose points are all farther apart than eps, but for a
few that were moved beside another; lists of three neighbours or of two.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture()
def lk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.get_device_properties(0).total_memory < (200 << 30):
        pytest.skip("needs the memory of an MI355X")
    from paper_2308_07173_amd import lkc
    ctx = lkc.Context()
    yield lkc, ctx
    ctx.close()
    torch.cuda.empty_cache()


def test_clustering_of_more_than_2_27_points(lk):
    """32 lanes a point would be 2^32 threads from 2^27 points on."""
    lkc, ctx = lk
    n = (1 << 27) + 77
    i = torch.arange(n, device="cuda", dtype=torch.int32)
    p = torch.empty(n, 3, device="cuda")
    p[:, 0] = i % 4096
    p[:, 1] = torch.div(i, 4096, rounding_mode="floor") % 4096
    p[:, 2] = torch.div(i, 1 << 24, rounding_mode="floor")
    near = {n - 1: 5, n - 40: (1 << 26) + 3, (1 << 26): (1 << 26) - 1, 1 << 20: 7}
    want = i.clone()
    for a, b in near.items():
        p[a] = p[b] + torch.tensor([0.25, 0.0, 0.0], device="cuda")
        want[a] = b
    del i
    labels, k = lkc.lkc_euclid_cluster(ctx, p, 0.5)
    assert k == n - len(near)
    assert torch.equal(labels, want)
    del labels
    for _ in range(2):
        out = lkc.lkc_euclid_cluster_async(ctx, p, 0.5)
        assert int(out["status"]) == 0 and int(out["n_clusters"]) == n - len(near)
        assert torch.equal(out["labels"], want)
        del out


def test_covariances_of_more_than_2_30_lists(lk):
    """256 threads for 64 lists would be 2^32 threads from 2^30 lists on."""
    lkc, ctx = lk
    p = torch.tensor([[0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1]], dtype=torch.float32).cuda()
    t = lkc.lkc_build_target(ctx, p, 1.0)
    q = (1 << 30) + 131
    idx = torch.tensor([[0, 1, 2]], dtype=torch.int32, device="cuda").repeat(q, 1)
    cnt = torch.full((q,), 3, dtype=torch.int32, device="cuda")
    few = [0, 63, 64, (1 << 30) - 1, 1 << 30, (1 << 30) + 63, q - 1]
    cnt[few] = 2
    out = dict(mean=None, cov=None, reg=None,
               valid=torch.full((q,), 7, dtype=torch.uint8, device="cuda"))
    lkc.lkc_covariances(ctx, t, idx, cnt, plane_eps=1e-3, out=out)
    torch.cuda.synchronize()
    assert not out["valid"][few].any()
    out["valid"][few] = 1
    assert bool((out["valid"] == 1).all())
    t.free()
