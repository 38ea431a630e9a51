"""The grid that lkc_euclid_cluster leaves in a context for the call without a
wait: laid out for the cloud and the eps of the last synchronous call, whatever
calls came before it."""
import numpy as np
import pytest

from paper_2308_07173_amd import workloads
from tests import parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# 8-bit sort passes that a grid of 0.375 m cells takes, with 2 bits a cell axis
# below the cell key: 2 (6 cells an axis), 3 (24; the cell key alone fits 2), 3 (107)
SMALL, MID, LARGE = 2.0, 9.0, 40.0


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


@pytest.mark.parametrize("n", [3000, 12000])
@pytest.mark.parametrize("before", [[SMALL, MID], [SMALL, SMALL, MID, MID], [4000.0, SMALL, MID]])
def test_passes_of_the_last_synchronous_call(n, before):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_07173_amd import lkc
    ctx = lkc.Context()
    for i, side in enumerate(before):
        p = workloads.random_cloud(n, i, scale=side / 2)
        labels, k = lkc.lkc_euclid_cluster(ctx, dev(p), 0.3)
        if i == len(before) - 1:
            parity.check_clusters(p, 0.3, labels.cpu().numpy(), k)
    large = workloads.random_cloud(n, 9, scale=LARGE / 2)
    out = lkc.lkc_euclid_cluster_async(ctx, dev(large), 0.3)
    assert int(out["status"]) == lkc.LKC_OK
    parity.check_clusters(large, 0.3, out["labels"].cpu().numpy(), int(out["n_clusters"]))
    ctx.close()


def test_more_passes_do_not_outlive_the_cloud_that_needed_them():
    """Three passes' worth of cloud, then two: the call without a wait finds
    the second's grid, and a cloud past it is refused as after any such call."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_07173_amd import lkc
    ctx = lkc.Context()
    small, large = (workloads.random_cloud(3000, 1, scale=s / 2) for s in (SMALL, LARGE))
    lkc.lkc_euclid_cluster(ctx, dev(large), 0.3)
    for _ in range(2):
        lkc.lkc_euclid_cluster(ctx, dev(small), 0.3)
    out = lkc.lkc_euclid_cluster_async(ctx, dev(large), 0.3)
    assert int(out["status"]) == lkc.LKC_ERR_UNSUPPORTED
    lkc.lkc_euclid_cluster(ctx, dev(large), 0.3)
    out = lkc.lkc_euclid_cluster_async(ctx, dev(large), 0.3)
    assert int(out["status"]) == lkc.LKC_OK
    ctx.close()
