"""The LBVH traversal's groups of 64 leaves and the brute-force tiles against the oracle's
candidates: sizes around a group, a tree level and a tile; groups that straddle problems; groups
whose box spans the scene; searches handed over at a low budget; boxes beyond float32's range."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _soup(seed, n, spread=1.0, size=0.15, pool=None):
    """n triangles on a pool of random points near their centres (shared vertices included)."""
    rng = np.random.default_rng(seed)
    pool = pool or max(4, n)
    c = rng.uniform(0.0, spread, (pool, 3))
    tris = np.empty((n, 3), np.int32)
    near = np.argsort(((c[:, None, :] - c[None, :256, :]) ** 2).sum(-1) if pool <= 512 else rng.random((pool, 8)), axis=1)
    for k in range(n):
        v = rng.integers(0, pool)
        tris[k] = (v, *(near[v, rng.permutation(min(8, near.shape[1]))[:2]] if pool <= 512 else rng.integers(0, pool, 2)))
    x = c + rng.normal(0.0, 1e-3, c.shape)
    if pool > 512:  # separate corners around each triangle's centre
        x = (rng.uniform(0.0, spread, (n, 1, 3)) + rng.normal(0.0, size, (n, 3, 3))).reshape(-1, 3)
        tris = np.arange(3 * n, dtype=np.int32).reshape(n, 3)
    return np.ascontiguousarray(x), np.ascontiguousarray(tris)


def _pairs(x, tris, method, budget=0, capacity=None):
    import torch

    from paper_2606_06511_amd import ttie

    ref = oracle.pairs(x, tris) if method != ttie.BROAD_BRUTE else None
    n_ref = len(ref) if ref is not None else len(tris) * (len(tris) - 1) // 2
    ctx = ttie.Context(0)
    cap = capacity or max(n_ref, 1)  # no slot to spare
    ctx.reserve(len(x), len(tris), cap, max_hits=64)
    ctx.set_param(ttie.PARAM_TRAV_BUDGET, budget)
    p, n = ctx.broadphase(torch.from_numpy(x).cuda(), torch.from_numpy(tris).cuda(), method, capacity=cap)
    assert ctx.status() == ttie.TTIE_OK
    got = p[: int(n.item())].cpu().numpy()
    return got[np.lexsort((got[:, 1], got[:, 0]))], ref


@pytest.mark.parametrize("n", [2, 3, 5, 15, 17, 63, 64, 65, 127, 129, 255, 257, 1023, 1025, 4095, 4097, 16390])
def test_group_sizes(n):
    from paper_2606_06511_amd import ttie

    x, tris = _soup(n, n, spread=max(1.0, (n / 64) ** (1 / 3)))
    got, ref = _pairs(x, tris, ttie.BROAD_LBVH)
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("n", [2, 15, 16, 17, 255, 256, 257, 300, 1000])
def test_brute_tiles(n):
    from paper_2606_06511_amd import ttie

    x, tris = _soup(n, n, pool=max(4, n // 2))
    got, _ = _pairs(x, tris, ttie.BROAD_BRUTE)
    i, j = np.triu_indices(n, 1)
    keep = ~(tris[i][:, :, None] == tris[j][:, None, :]).any((1, 2))
    assert np.array_equal(got, np.stack([i[keep], j[keep]], 1))


@pytest.mark.parametrize("budget", [16, 0])
@pytest.mark.parametrize("kind", ["overlapping", "mixed_sizes", "clusters", "line"])
def test_loose_groups(kind, budget):
    """Groups that meet much of the scene: handed over at the low budget, nodes and candidates."""
    from paper_2606_06511_amd import ttie

    rng = np.random.default_rng(5)
    if kind == "overlapping":  # every box overlaps hundreds
        x, tris = _soup(1, 3000, spread=1.0, size=0.1, pool=600)
    elif kind == "mixed_sizes":  # a few huge triangles among small ones
        x, tris = _soup(2, 20000, spread=20.0, size=0.1, pool=600)
        big = rng.choice(20000, 40, replace=False)
        x = x.reshape(-1, 3, 3)
        x[big] = 10.0 + (x[big] - x[big].mean(1, keepdims=True)) * 100.0
        x = x.reshape(-1, 3)
    elif kind == "clusters":  # far apart: the curve jumps inside groups
        x, tris = _soup(3, 9000, spread=1.0, size=0.05, pool=600)
        x = (x.reshape(-1, 3, 3) + 1000.0 * rng.integers(0, 5, (9000, 1, 3))).reshape(-1, 3)
    else:  # all boxes flat in two axes
        x, tris = _soup(4, 3000, spread=50.0, size=0.1, pool=600)
        x[:, 1:] = 0.25
    got, ref = _pairs(np.ascontiguousarray(x), tris, ttie.BROAD_LBVH, budget)
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("scale", [2.0**-150, 2.0**130, 2.0**190])
def test_beyond_float32(scale):
    from paper_2606_06511_amd import ttie

    x, tris = _soup(7, 700, spread=3.0, size=0.2, pool=600)
    x = x - 1.5
    x[::7] *= scale
    got, ref = _pairs(np.ascontiguousarray(x), tris, ttie.BROAD_LBVH)
    assert np.array_equal(got, ref)


def test_problems_inside_groups():
    """Many problems smaller than a group, all in the same place."""
    import torch

    from paper_2606_06511_amd import ttie, workloads

    probs = [_soup(100 + k, 1 + (7 * k) % 90, spread=1.0, size=0.2, pool=600) for k in range(60)]
    x, tris, _, tri_off = workloads.concat_problems(probs)
    ref = []
    vo = 0
    for k, (px, pt) in enumerate(probs):
        ref.append(oracle.pairs(px, pt) + tri_off[k] if len(pt) > 1 else np.zeros((0, 2), np.int64))
        vo += len(px)
    ref = np.concatenate(ref)
    ref = ref[np.lexsort((ref[:, 1], ref[:, 0]))]
    ctx = ttie.Context(0)
    ctx.reserve(len(x), len(tris), len(ref), max_hits=64)
    p, n = ctx.batch_broadphase(torch.from_numpy(x).cuda(), torch.from_numpy(tris).cuda(),
                                torch.from_numpy(tri_off).cuda())
    assert ctx.status() == ttie.TTIE_OK
    got = p[: int(n.item())].cpu().numpy()
    got = got[np.lexsort((got[:, 1], got[:, 0]))]
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("n,budget", [(524288, 16), (524288, 0), (524289, 16), (524289, 0), (1048577, 16), (1048577, 0)])
def test_both_handover_rules(n, budget):
    """On both sides of the sizes from which searches are handed over later, and taken up whole,
    against the candidates of the spatial hash; a tenth of the triangles in a dense heap, whose
    searches are over any budget."""
    import torch

    from paper_2606_06511_amd import ttie

    rng = np.random.default_rng(n)
    c = rng.uniform(0.0, 100.0, (n, 1, 3))
    c[: n // 10] = rng.uniform(0.0, 5.0, (n // 10, 1, 3))
    x = torch.from_numpy((c + rng.normal(0.0, 0.15, (n, 3, 3))).reshape(-1, 3)).cuda()
    tris = torch.arange(3 * n, dtype=torch.int32, device="cuda").reshape(n, 3)
    ctx = ttie.Context(0)
    cap = 16_000_000
    ctx.reserve(3 * n, n, cap, max_hits=64)
    ctx.set_param(ttie.PARAM_TRAV_BUDGET, budget)
    keys = []
    for method in (ttie.BROAD_HASH, ttie.BROAD_LBVH):
        p, k = ctx.broadphase(x, tris, method, capacity=cap)
        assert ctx.status() == ttie.TTIE_OK
        p = p[: int(k.item())].long()
        assert len(p) > n // 10
        keys.append(torch.sort(p[:, 0] * n + p[:, 1]).values)
    assert torch.equal(*keys)
