"""The voxel filters where their tiles of 2,048 sorted points can go wrong:
sizes at a tile's edges, voxels that fill or span several tiles, one voxel of
all points, points left out at the end, 32-bit and 64-bit keys, and more tiles
than add up their own counts.  Centroids are the float32 rounding of FP64 means
added in ascending point order: exact against the oracle.
"""
import numpy as np
import pytest

from oracle import oracle
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


def check(lk, p, leaf, axis_bits=None):
    lkc, ctx = lk
    d = torch.from_numpy(np.ascontiguousarray(p, np.float32)).cuda()
    o = oracle.voxel_filter(p, leaf)
    g = lkc.lkc_voxel_filter(ctx, d, leaf)
    outs = [{k: v.cpu().numpy() for k, v in g.items()}]
    if axis_bits:
        a = lkc.lkc_voxel_filter_async(ctx, d, leaf, axis_bits)
        m = int(a["n_out"])
        assert int(a["status"]) == 0
        outs.append({k: a[k][:m].cpu().numpy() for k in ("centroid", "count", "voxel")})
    for g in outs:
        assert np.array_equal(g["count"], o["count"])
        assert np.array_equal(g["voxel"], o["voxel"])
        assert np.array_equal(g["centroid"], o["centroid"].astype(np.float32))


@pytest.mark.parametrize("n", [1, 255, 256, 257, 2047, 2048, 2049, 4096, 6145])
@pytest.mark.parametrize("leaf", [0.05, 1.0, 100.0])
def test_tile_edges(lk, n, leaf):
    p = workloads.random_cloud(n, n, scale=4.0, offset=(50.0, -20.0, 3.0))
    check(lk, p, leaf, axis_bits=12)
    if n > 20:
        p[::7] = np.nan
        p[-3:] = np.inf
        check(lk, p, leaf, axis_bits=12)


@pytest.mark.parametrize("runs", [(2048, 2048, 1), (5000,), (1, 4095, 1, 2049, 300), (2047, 1, 2048),
                                  (2048 * 3 + 5, 2048 * 2 - 5, 2)])
def test_voxels_that_span_tiles(lk, runs):
    rng = np.random.default_rng(len(runs))
    at = np.repeat(np.arange(len(runs)), runs)
    p = rng.uniform(0.05, 0.95, (at.size, 3)) + np.stack([at, 0 * at, 0 * at], 1)
    p = p.astype(np.float32)[rng.permutation(at.size)]
    check(lk, p, 1.0, axis_bits=10)
    check(lk, p, 1.0, axis_bits=11)     # 34 key bits


def test_sparse_wide_box_takes_64_bit_keys(lk):
    p = workloads.random_cloud(9000, 4, scale=3000.0)
    check(lk, p, 0.02)


def test_more_tiles_than_add_up_their_counts(lk):
    n = 4096 * 2048 + 1000
    rng = np.random.default_rng(1)
    p = np.empty((n, 3), np.float32)
    p[:] = rng.random((n, 3), dtype=np.float32) * np.float32(40.0)
    p[:, 2] *= np.float32(0.05)
    check(lk, p, 0.5, axis_bits=7)
