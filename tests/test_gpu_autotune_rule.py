"""The autotuner's candidates that come to the same launch, and a sample that
the wavefront search would be fastest on though all queries would not."""
import numpy as np
import pytest

from paper_2308_07173_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("queries,cfgs,chosen,same", [
    (5_000, (dict(), dict(algorithm=2), dict(algorithm=2, waves_per_block=4)), dict(), True),
    (200_000, (dict(algorithm=2), dict()), dict(), False),
    (200_000, (dict(algorithm=2),), dict(algorithm=2), True),
])
def test_candidates_by_the_search_all_queries_take(queries, cfgs, chosen, same):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_07173_amd import autotune, lkc
    ctx = lkc.Context()
    p = workloads.plane_wall(20_000, seed=3)
    q = np.tile(p, (10, 1))[:queries]
    r = autotune.autotune(p, q, 10, 1.0, cells=(1.0,), cfgs=cfgs, sample=2_000, ctx=ctx)
    assert r["cfg"] == chosen and r["cell"] == 1.0 and r["sample"] == 2_000
    times = [ms for _, _, ms in r["table"]]
    assert all(ms > 0 for ms in times)
    assert (len(set(times)) == 1) == same
    assert r["ms"] == times[[dict(c) for c in cfgs].index(chosen)]
    ctx.close()
