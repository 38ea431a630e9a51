"""Clustering where its passes can go wrong: chains far longer than a hook
reaches, in every index order; mask tiles of 1,024 at their edges; a grid that
a second call rebuilds without a wait, in its old sort passes or past them, and
a cloud that such a rebuild has to refuse.  Chains and lattices have one right
answer in float32; random clouds follow the boundary-band rule of
``tests/parity.py``.
"""
import numpy as np
import pytest

from paper_2308_07173_amd import workloads
from tests import parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture()
def lk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_07173_amd import lkc
    ctx = lkc.Context()
    yield lkc, ctx
    ctx.close()


def dev(a, dtype=np.float32):
    return torch.from_numpy(np.ascontiguousarray(a, dtype)).cuda()


def chain(n, order, seed=0):
    p = np.zeros((n, 3), np.float32)
    p[:, 0] = np.arange(n) * np.float32(0.25)
    if order == "down":
        p = p[::-1]
    elif order == "random":
        p = p[np.random.default_rng(seed).permutation(n)]
    elif order == "ends":      # neighbours far apart in index
        p = np.concatenate([p[::2], p[1::2][::-1]])
    return p.copy()


@pytest.mark.parametrize("order", ["up", "down", "random", "ends"])
@pytest.mark.parametrize("n", [1, 2, 65, 4097, 30011])
def test_chains_and_gaps(lk, n, order):
    lkc, ctx = lk
    p = chain(n, order)
    for _ in range(2):
        labels, k = lkc.lkc_euclid_cluster(ctx, dev(p), 0.25)
        assert k == 1 and not labels.any()
    gap = p[:, 0] >= np.float32(0.25 * (n // 2))
    q = p.copy()
    q[gap, 0] += 100.0
    want = np.where(gap, np.flatnonzero(gap).min() if gap.any() else 0,
                    np.flatnonzero(~gap).min() if (~gap).any() else 0)
    for call in (lkc.lkc_euclid_cluster, lkc.lkc_euclid_cluster_async):
        r = call(ctx, dev(q), 0.25)
        labels = r[0] if isinstance(r, tuple) else r["labels"]
        assert np.array_equal(labels.cpu().numpy(), want)


@pytest.mark.parametrize("n", [1023, 1024, 1025, 4097, 12289])
def test_mask_tiles(lk, n):
    lkc, ctx = lk
    rng = np.random.default_rng(n)
    p = workloads.random_cloud(n, n, scale=6.0)
    for share in (0.0, 0.02, 0.9, 1.0):
        mask = (rng.random(n) < share).astype(np.uint8)
        labels, k = lkc.lkc_euclid_cluster(ctx, dev(p), 0.4, mask=dev(mask, np.uint8))
        labels = labels.cpu().numpy()
        kept = np.flatnonzero(mask)
        assert (labels[mask == 0] == -1).all()
        if kept.size:
            back = np.full(n, -1)
            back[kept] = np.arange(kept.size)
            parity.check_clusters(p[kept], 0.4, back[labels[kept]], k)
        else:
            assert k == 0


def test_second_call_on_the_grid_of_the_first(lk):
    lkc, ctx = lk
    small = workloads.random_cloud(3000, 5, scale=3.0)
    wide = workloads.random_cloud(3000, 6, scale=3.0)
    wide[::3] += np.array([30000.0, -20000.0, 9000.0], np.float32)   # more sort passes
    bad = small.copy()
    bad[1234, 1] = np.inf
    for cloud, eps in ((small, 0.3), (small, 0.3), (wide, 0.3), (small, 0.5), (wide, 0.2)):
        labels, k = lkc.lkc_euclid_cluster(ctx, dev(cloud), eps)
        parity.check_clusters(cloud, eps, labels.cpu().numpy(), k)
    with pytest.raises(lkc.LkcError) as e:
        lkc.lkc_euclid_cluster(ctx, dev(bad), 0.3)
    assert e.value.status == lkc.LKC_ERR_NONFINITE
    with pytest.raises(lkc.LkcError) as e:
        lkc.lkc_euclid_cluster(ctx, dev(wide), 0.02)
    assert e.value.status == lkc.LKC_ERR_INVALID_ARG
    labels, k = lkc.lkc_euclid_cluster(ctx, dev(small), 0.3)
    parity.check_clusters(small, 0.3, labels.cpu().numpy(), k)
    out = lkc.lkc_euclid_cluster_async(ctx, dev(bad), 0.3)
    assert int(out["status"]) == lkc.LKC_ERR_NONFINITE and int(out["n_clusters"]) == 0
