"""lkc_covariances where its workgroups' rows end: query counts around their
sizes, the shortest and longest lists, lists cut by an entry that names no
point.  The fused search's covariances (checked against the oracle elsewhere)
must come out in the same bits."""
import numpy as np
import pytest

from paper_2308_07173_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("k", [1, 2, 20, 45, 64])
@pytest.mark.parametrize("q", [1, 15, 64, 65, 1000])
@pytest.mark.parametrize("kernel", ["none", "gaussian"])
def test_cut_lists_and_remainders(k, q, kernel):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_07173_amd import lkc
    ctx = lkc.Context()
    p = workloads.plane_wall(3000, seed=8)
    t = lkc.lkc_build_target(ctx, torch.from_numpy(p).cuda(), 1.0)
    qd = torch.from_numpy(workloads.random_cloud(q, 9, scale=8.0)).cuda()
    f = lkc.lkc_knn_cov_weighted(ctx, t, qd, k, kernel, 0.4, 2.5)

    def cov(idx, cnt, queries):
        return lkc.lkc_covariances_weighted(ctx, t, idx, cnt, kernel, 0.4, queries=queries)

    full = cov(f["idx"], f["count"], qd)
    for key in ("mean", "cov", "reg", "valid"):
        assert torch.equal(full[key], f[key]), key
    # cut by the count, and by an entry outside the target
    rng = np.random.default_rng(k * 1000 + q)
    cut = torch.from_numpy(rng.integers(0, k + 1, q).astype(np.int32)).cuda()
    cnt = torch.minimum(cut, f["count"])
    for bad in (-1, 3000, 2**31 - 1):
        idx = f["idx"].clone()
        rows = torch.nonzero(cut < k).flatten()
        idx[rows, cut[rows].long()] = bad
        for queries in (qd, None):
            a = cov(f["idx"], cnt, queries)
            b = cov(idx, f["count"], queries)
            for key in a:
                assert torch.equal(a[key], b[key]), (key, bad)
    t.free()
    ctx.close()
