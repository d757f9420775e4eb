"""Batches of problems smaller than the traversal's groups, all in one place, so that every group
overlaps itself across its problems' borders."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _batch(sizes, spread=0.0):
    from paper_2606_06511_amd import workloads

    rng = np.random.default_rng(len(sizes))
    probs = []
    for n in sizes:
        c = rng.uniform(0.0, 1.0, (n, 1, 3)) + spread * rng.normal(size=3)
        probs.append(((c + rng.normal(0.0, 0.3, (n, 3, 3))).reshape(-1, 3), np.arange(3 * n, dtype=np.int32).reshape(n, 3)))
    x, tris, _, tri_off = workloads.concat_problems(probs)
    return probs, x, tris, tri_off


@pytest.mark.parametrize("sizes", [[1] * 200, [2] * 100, [8] * 60, [7, 9] * 40, [15, 16, 17] * 12, list(range(1, 70)),
                                   [63, 64, 65, 1, 128, 3], [100, 1, 1, 1, 61, 30, 200, 5]], ids=lambda s: f"{len(s)}x{s[0]}")
def test_pairs_stay_in_their_problem(sizes):
    import torch

    from paper_2606_06511_amd import ttie

    probs, x, tris, tri_off = _batch(sizes)
    ref = np.concatenate([oracle.pairs(px, pt) + tri_off[k] if len(pt) > 1 else np.zeros((0, 2), np.int64)
                          for k, (px, pt) in enumerate(probs)])
    ref = ref[np.lexsort((ref[:, 1], ref[:, 0]))]
    ctx = ttie.Context(0)
    ctx.reserve(len(x), len(tris), max(len(ref), 1), max_hits=64)
    p, n = ctx.batch_broadphase(*[torch.from_numpy(a).cuda() for a in (x, tris, tri_off)])
    assert ctx.status() == ttie.TTIE_OK
    got = p[: int(n.item())].cpu().numpy()
    assert np.array_equal(got[np.lexsort((got[:, 1], got[:, 0]))], ref)


def test_problems_in_one_place_cost_what_they_cost_apart():
    """1000 problems of 8 triangles: the traversal's time in one place and far apart (2.3 times as
    long where the overlaps across problems were listed and tested)."""
    import torch

    from paper_2606_06511_amd import ttie

    best = []
    for spread in (100.0, 0.0):
        _, x, tris, tri_off = _batch([8] * 1000, spread)
        dev = [torch.from_numpy(a).cuda() for a in (x, tris, tri_off)]
        ctx = ttie.Context(0)
        ctx.reserve(len(x), len(tris), 1 << 17, max_hits=64)
        out = ctx.batch_broadphase(*dev)
        ctx.check()
        ctx.set_timing(["bp_traverse"])
        ms = []
        for _ in range(20):
            ctx.batch_broadphase(*dev, out=out)
            ctx.check()
            ms.append(ctx.read_timers()["bp_traverse"][1])
        best.append(min(ms))
    assert best[1] < 1.7 * best[0], best
