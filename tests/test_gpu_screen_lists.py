"""Candidates left to the exact pass travel in the screening's lists and are gathered by waves:
few and many of them, scattered and in runs longer than a wave's buffer, against the oracle's flags
and hit count."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _nearly_coplanar(seed=0, n=10):
    """Two rotated, nearly coincident planar grids crossed by a third: most pairs of the first two
    are within the filter's bound of being coplanar."""
    from paper_2606_06511_amd import workloads

    rng = np.random.default_rng(seed)
    q, _ = np.linalg.qr(rng.normal(size=(3, 3)))
    x, t = workloads.grid_mesh(n)
    a = x - 0.5
    b = a + np.array([0.5 / (n - 1), 0.3 / (n - 1), 0.0])
    b[:, 2] += 2.0**-52 * rng.integers(-2, 3, len(b))
    c = a[:, [0, 2, 1]] * 0.9 + np.array([0.0, 0.01, 0.01])
    xs = np.concatenate([a @ q.T, b @ q.T, c @ q.T])
    return np.ascontiguousarray(xs), np.ascontiguousarray(np.concatenate([t, t + n * n, t + 2 * n * n]).astype(np.int32))


@pytest.mark.parametrize("tile", [0, 256])
@pytest.mark.parametrize("how", ["once", "few", "tiled", "runs"])
def test_deferred_lists(how, tile):
    import torch

    from paper_2606_06511_amd import ttie

    x, tris = _nearly_coplanar()
    pairs = oracle.pairs(x, tris).astype(np.int32)
    rng = np.random.default_rng(1)
    if how == "few":
        pairs = pairs[rng.permutation(len(pairs))[:37]]
    elif how == "tiled":
        pairs = np.tile(pairs, (60, 1))
    elif how == "runs":
        pairs = np.repeat(pairs, 700, axis=0)[: 1 << 18]
    uniq, inv = np.unique(pairs, axis=0, return_inverse=True)
    ref = oracle.evaluate(x, tris, uniq, hessian=False)["flags"][inv.reshape(-1)]
    n_hits = int(((ref == 1) | (ref == 3)).sum())
    ctx = ttie.Context(0)
    ctx.reserve(len(x), len(tris), len(pairs), max_hits=max(n_hits, 64))
    ctx.set_param(ttie.PARAM_SCREEN_TILE, tile)
    out = ctx.evaluate(torch.from_numpy(x).cuda(), torch.from_numpy(tris).cuda(),
                       torch.from_numpy(np.ascontiguousarray(pairs)).cuda(), hessian=False, flags=True)
    ctx.check()
    assert np.array_equal(out["flags"].cpu().numpy(), ref)
    assert int(out["n_hits"].item()) == int((ref == 1).sum())


@pytest.mark.parametrize("blocks", [0, 64])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 64 * 256 - 1, 64 * 256 + 1, 3 * 64 * 256 + 63, 64 * 6144 - 1, 64 * 6144 + 65])
def test_chunks_of_the_list(n, blocks):
    """Lists around a batch of 64 and around a batch for each of the grid's waves (256 with 64
    blocks, 6,144 by default), which take one batch more or less than each other."""
    import torch

    from paper_2606_06511_amd import ttie, workloads

    x, tris = workloads.folded_cloth(2, n=64)
    pairs = oracle.pairs(x, tris).astype(np.int32)
    ref = oracle.evaluate(x, tris, pairs, hessian=False)["flags"]
    take = np.random.default_rng(n).integers(0, len(pairs), n)
    ctx = ttie.Context(0)
    ctx.reserve(len(x), len(tris), n, max_hits=max(64, int((ref[take] == 1).sum())))
    ctx.set_param(ttie.PARAM_SCREEN_BLOCKS, blocks)
    out = ctx.evaluate(torch.from_numpy(x).cuda(), torch.from_numpy(tris).cuda(),
                       torch.from_numpy(pairs[take]).cuda(), hessian=False, flags=True)
    ctx.check()
    assert np.array_equal(out["flags"].cpu().numpy(), ref[take])
    assert int(out["n_hits"].item()) == int((ref[take] == 1).sum())


@pytest.mark.parametrize("capacity", [1 << 24, (1 << 24) + 1])
def test_both_grids(capacity):
    """On both sides of the pair capacity at which the screening's grid changes."""
    import torch

    from paper_2606_06511_amd import ttie, workloads

    x, tris = workloads.folded_cloth(2, n=64)
    pairs = oracle.pairs(x, tris)
    ref = oracle.evaluate(x, tris, pairs, hessian=False)
    ctx = ttie.Context(0)
    ctx.reserve(len(x), len(tris), capacity, max_hits=1 << 12)
    buf = torch.zeros((capacity, 2), dtype=torch.int32, device="cuda")
    buf[: len(pairs)] = torch.from_numpy(pairs.astype(np.int32)).cuda()
    out = ctx.evaluate(torch.from_numpy(x).cuda(), torch.from_numpy(tris).cuda(), buf,
                       torch.tensor([len(pairs)], device="cuda"), hessian=False, flags=True)
    ctx.check()
    assert np.array_equal(out["flags"][: len(pairs)].cpu().numpy(), ref["flags"])
    assert int(out["n_hits"].item()) == len(ref["hit_pair"]) > 0
