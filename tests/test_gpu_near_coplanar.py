"""Pairs whose plane sides are within the float64 filter's bound but (mostly) not zero: triangles
of rotated planes, whose corners lie off the plane by their rounding, alone and lifted by a few
units in the last place, and crossing pairs among them.  Flags and hits against the oracle's
exact decisions (the line of two nearly equal planes, and T with it, has no accurate float64
value)."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _planes(seed, lift, n=14):
    """Two rotated planar grids in one plane (the second shifted by half a cell and lifted by
    `lift` units of 2^-52), crossed by a third grid that contains one of their edges' lines."""
    rng = np.random.default_rng(seed)
    from paper_2606_06511_amd import workloads

    q, _ = np.linalg.qr(rng.normal(size=(3, 3)))
    x, t = workloads.grid_mesh(n)
    a = x - 0.5
    b = a + np.array([0.5 / (n - 1), 0.3 / (n - 1), 0.0])
    b[:, 2] += lift * 2.0**-52 * rng.integers(-2, 3, len(b))
    c = a[:, [0, 2, 1]] * 0.9 + np.array([0.0, 0.5 / (n - 1) * rng.integers(0, 3), 0.01])
    xs = np.concatenate([a @ q.T, b @ q.T, c @ q.T]) * 10.0 ** rng.integers(-3, 4)
    return np.ascontiguousarray(xs), np.ascontiguousarray(np.concatenate([t, t + n * n, t + 2 * n * n]).astype(np.int32))


@pytest.mark.parametrize("lift", [0, 1, 50])
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_near_coplanar_flags(seed, lift):
    import torch

    from paper_2606_06511_amd import ttie

    x, tris = _planes(seed, lift)
    pairs = oracle.pairs(x, tris)
    ref = oracle.evaluate(x, tris, pairs)
    ctx = ttie.Context(0)
    ctx.reserve(len(x), len(tris), len(pairs), max_hits=len(pairs))
    dev = torch.device("cuda", 0)
    out = ctx.evaluate(torch.from_numpy(x).to(dev), torch.from_numpy(tris).to(dev),
                       torch.from_numpy(pairs.astype(np.int32)).to(dev).contiguous(), flags=True)
    ctx.check()
    assert np.array_equal(out["flags"].cpu().numpy(), ref["flags"])
    assert int(out["n_hits"].item()) == len(ref["hit_pair"]) > 0
