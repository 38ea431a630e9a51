"""The order in which the group search takes its queries: by target, then by
the Morton code of their cell (an axis dropping out above its own bits) and
sub-cell, equal keys as they came.  The order does not show in the results, but
in how many of a group's lanes lie near its anchor, which the profile counts:
worked out here from the keys' definition, group by group."""
import numpy as np
import pytest

from paper_2308_07173_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BOXES = [(9, 9, 9), (60, 40, 1), (1, 300, 40), (40, 1, 300), (3000, 1, 1), (1, 1, 3000),
         (1500, 1500, 1500), (5, 700, 90)]
REACH = 2   # cells around an anchor


def cells_of(x, inv):
    return np.floor(x * inv).astype(np.int64)


def interleave(v, w):
    key = np.zeros(len(v), np.uint64)
    at = 0
    for level in range(max(w)):
        for a in range(3):
            if level < w[a]:
                key |= ((v[:, a] >> np.uint64(level)) & np.uint64(1)) << np.uint64(at)
                at += 1
    return key


def members(targets, q, tgt):
    """Lanes of every 64-query group that its one round searches for; `targets`
    [(cell size, box min, box max)] in cells."""
    ext = np.stack([hi - lo + 2 for _, lo, hi in targets]).max(axis=0)
    w = [max(1, int(e).bit_length()) for e in ext]
    tbits = (len(targets) - 1).bit_length()
    lo2 = max(0, min(2, (63 - tbits - sum(w)) // 3))
    room = min(63, 8 * ((tbits + sum(w) + 3 * lo2 + 7) // 8)) - tbits
    sub = max(lo2, min(4, (room - sum(w)) // 3))
    shift = sum(w) + 3 * sub
    assert shift + tbits <= 63
    cell, v = np.zeros((len(q), 3), np.int64), np.zeros((len(q), 3), np.uint64)
    for t, (size, lo, hi) in enumerate(targets):
        on = tgt == t
        inv = np.float32(1.0) / np.float32(size)
        u = q[on] * inv
        c = np.floor(u).astype(np.int64)
        s = np.clip(((u - np.floor(u)) * np.float32(1 << sub)).astype(np.int64), 0, (1 << sub) - 1)
        cl = np.clip(c - (lo - 1), 0, np.maximum(hi - lo, 0) + 2)
        cell[on] = c
        v[on] = ((cl << sub) | s).astype(np.uint64)
    key = interleave(v, [b + sub for b in w]) | (tgt.astype(np.uint64) << np.uint64(shift))
    order = np.argsort(key, kind="stable")
    out = []
    for g in range(0, len(q), 64):
        i = order[g:g + 64]
        same = tgt[i] == tgt[i[0]]
        c = cell[i][same]
        near = lambda a: int((np.abs(c - a) <= REACH).all(axis=1).sum())
        best = near(c[0])
        best = max(best, near(c[-1]), near((c.min(axis=0) + c.max(axis=0)) >> 1))
        out.append(best)
    return np.array(out)


def queries(box, n, seed):
    """In clusters a few cells wide, anywhere in a box (and just outside)."""
    rng = np.random.default_rng(seed)
    at = rng.uniform(-1.05, 1.05, (max(1, n // 300), 3)) * np.asarray(box)
    spread = np.minimum(3.0, np.asarray(box))
    return (at[rng.integers(0, len(at), n)] + rng.normal(0, 1, (n, 3)) * spread).astype(np.float32)


def build(lkc, ctx, box, n, seed, cell):
    p = (workloads.random_cloud(n, seed) * np.asarray(box, np.float32)).astype(np.float32)
    t = lkc.lkc_build_target(ctx, torch.from_numpy(p).cuda(), cell)
    i = t.info()
    return t, (cell, np.array(i["cell_min"]), np.array(i["cell_max"]))


@pytest.mark.parametrize("q_n", [3000, 200_001])
@pytest.mark.parametrize("box", BOXES)
def test_one_target(box, q_n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_07173_amd import lkc
    ctx = lkc.Context()
    t, d = build(lkc, ctx, box, 6000, 7, 0.5)
    q = queries(box, q_n, 8)
    words = torch.zeros((q_n + 63) // 64, 25, dtype=torch.int32, device="cuda")
    ctx.set_profile(words)
    lkc.lkc_knn_query(ctx, t, torch.from_numpy(q).cuda(), 5, 1.0, cfg=dict(algorithm=1))
    got = words.cpu().numpy()[:, 6]
    ctx.set_profile(None)
    assert np.array_equal(got, members([d], q, np.zeros(q_n, np.int64)))
    t.free()
    ctx.close()


@pytest.mark.parametrize("boxes", [BOXES[:2], BOXES[1:4], BOXES[4:6] + BOXES[:1], BOXES[2:7]])
def test_several_targets(boxes):
    """64-bit keys with the target above them; boxes of different shapes share
    the widths of the widest."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_07173_amd import lkc
    ctx = lkc.Context()
    made = [build(lkc, ctx, b, 5000 + i, i, (0.5, 1.0, 0.75)[i % 3]) for i, b in enumerate(boxes)]
    scans, parts, tgt, at = [], [], [], 0
    for i in range(9):
        w, n = (i * 2) % len(boxes), (700, 1, 1300, 64, 2000)[i % 5]
        parts.append(queries(boxes[w], n, 20 + i))
        tgt.append(np.full(n, w))
        scans.append((at, n, w))
        at += n
    q, tgt = np.concatenate(parts).astype(np.float32), np.concatenate(tgt)
    ts = lkc.TargetSet(ctx, [m[0] for m in made], 16)
    ts.stage(scans)
    words = torch.zeros((at + 63) // 64, 25, dtype=torch.int32, device="cuda")
    ctx.set_profile(words)
    got = lkc.lkc_knn_cov_batched(ctx, ts, torch.from_numpy(q).cuda(), 6, 2.0, 1e-3,
                                  cfg=dict(algorithm=1))
    n_members = words.cpu().numpy()[:, 6]
    ctx.set_profile(None)
    assert np.array_equal(n_members, members([m[1] for m in made], q, tgt))
    wave = lkc.lkc_knn_cov_batched(ctx, ts, torch.from_numpy(q).cuda(), 6, 2.0, 1e-3,
                                   cfg=dict(algorithm=2))
    for key in got:
        assert torch.equal(got[key], wave[key]), key
    for (o, n, w) in scans:
        alone = lkc.lkc_knn_cov(ctx, made[w][0], torch.from_numpy(q[o:o + n]).cuda(), 6, 2.0, 1e-3)
        for key in alone:
            assert torch.equal(got[key][o:o + n], alone[key]), key
    ts.free()
    for m in made:
        m[0].free()
    ctx.close()
