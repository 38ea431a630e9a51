"""The group search's profile words (lkc_ctx_set_profile): cleared before every
search, also before one that the group search takes no part in."""
import numpy as np
import pytest

from paper_2308_07173_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("then", [dict(algorithm=2), None])
def test_words_of_the_search_before_do_not_stay(then):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_07173_amd import lkc
    ctx = lkc.Context()
    p = torch.from_numpy(workloads.plane_wall(6000, seed=1)).cuda()
    q = p[:3000].contiguous()
    t = lkc.lkc_build_target(ctx, p, 1.0)
    words = torch.full((47, 25), 5, dtype=torch.int32, device="cuda")
    ctx.set_profile(words)
    a = lkc.lkc_knn_cov(ctx, t, q, 10, 2.0, 1e-3, cfg=dict(algorithm=1))
    w = words.cpu().numpy()
    assert (w[:, 0] > 0).all() and w[:, 6].sum() + w[:, 7].sum() >= 3000
    b = lkc.lkc_knn_cov(ctx, t, q, 10, 2.0, 1e-3, cfg=then)
    assert not words.cpu().numpy().any()
    ctx.set_profile(None)
    for key in a:
        assert torch.equal(a[key], b[key]), key
    t.free()
    ctx.close()
