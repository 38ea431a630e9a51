"""A target whose box is too large for the query sort keys (2^21 cells an
axis).  A search that may sort its queries is refused, whatever their number;
the wavefront-per-query search, asked for, needs no keys and answers."""
import numpy as np
import pytest

from oracle import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("q", [1, 300, 99_000])
def test_refused_for_every_number_of_queries(q):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_07173_amd import lkc
    ctx = lkc.Context()
    lo, hi = -float(1 << 20), float((1 << 20) - 1)
    rng = np.random.default_rng(0)
    p = rng.uniform(-4, 4, (200, 3))
    p[0], p[1] = lo, hi
    p = p.astype(np.float32)
    t = lkc.lkc_build_target(ctx, torch.from_numpy(p).cuda(), 1.0)
    assert t.info()["cell_min"] == [-(1 << 20)] * 3 and t.info()["cell_max"] == [(1 << 20) - 1] * 3
    qs = rng.uniform(-4, 4, (q, 3)).astype(np.float32)
    qd = torch.from_numpy(qs).cuda()
    eye = torch.eye(3, device="cuda")
    calls = [
        lambda cfg: lkc.lkc_knn_query(ctx, t, qd, 5, 1.0, cfg=cfg),
        lambda cfg: lkc.lkc_knn_cov(ctx, t, qd, 5, 1.0, 1e-3, cfg=cfg),
        lambda cfg: lkc.lkc_knn_cov_weighted(ctx, t, qd, 5, "rbf", 1.0, 1.0, 1e-3, cfg=cfg),
        lambda cfg: lkc.lkc_gicp_linearize(ctx, t, eye.repeat(200, 1, 1), qd, eye.repeat(q, 1, 1),
                                           np.eye(4), 1.0, cfg=cfg),
    ]
    for call in calls:
        for cfg in (None, dict(algorithm=1)):
            with pytest.raises(lkc.LkcError) as e:
                call(cfg)
            assert e.value.status == lkc.LKC_ERR_UNSUPPORTED
        call(dict(algorithm=2))
    idx, d2, cnt = calls[0](dict(algorithm=2))
    rows = slice(0, 200)
    o_idx, _, o_cnt = oracle.knn(p, qs[rows], 5, 1.0)
    assert np.array_equal(cnt.cpu().numpy()[rows], o_cnt)
    # (a list longer than the group search takes was never sorted for it)
    lkc.lkc_knn_query(ctx, t, qd, 40, 1.0)
    t.free()
    ctx.close()


def test_autotune_is_refused_as_its_candidates_are():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_07173_amd import autotune, lkc
    ctx = lkc.Context()
    p = np.zeros((64, 3), np.float32)
    p[0], p[1] = -float(1 << 20), float((1 << 20) - 1)
    q = np.zeros((200, 3), np.float32)
    with pytest.raises(lkc.LkcError) as e:
        autotune.autotune(p, q, 5, 1.0, cells=(1.0,), ctx=ctx)
    assert e.value.status == lkc.LKC_ERR_UNSUPPORTED
    r = autotune.autotune(p, q, 5, 1.0, cells=(1.0,), cfgs=(dict(algorithm=2),), ctx=ctx)
    assert r["cfg"]["algorithm"] == 2
    ctx.close()
