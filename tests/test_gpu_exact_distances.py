"""Pairs that cross at a good angle with one vertex of either triangle a few units in the last place
off the other's plane: its sign is left to the exact pass, which takes the vertex's distance
afterwards, and the interval, T and the derivatives have accurate values to compare with."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

U = 2.0**-53


def _uncertain(a, b, c, p):
    """Whether p's side of the plane (a, b, c) is within the float64 filter's bound (9 u perm) by a
    factor of two."""
    e1, e2, w = b - a, c - a, p - a
    det = np.dot(np.cross(e1, e2), w)
    n = np.array([abs(e1[(k + 1) % 3] * e2[(k + 2) % 3]) + abs(e1[(k + 2) % 3] * e2[(k + 1) % 3]) for k in range(3)])
    return abs(det) <= 4.5 * U * np.dot(n, np.abs(w))


def _pairs_near(vertex, lift, n, seed):
    """n pairs; vertex k of the first triangle (k < 3) or k - 3 of the second lies near the other's
    plane, inside it, and the other two on either side of it."""
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < n:
        q, _ = np.linalg.qr(rng.normal(size=(3, 3)))
        base = np.array([[-1.0, -0.8, 0.0], [1.2, -0.7, 0.0], [0.1, 1.1, 0.0]]) + np.append(rng.uniform(-0.1, 0.1, 2), 0.0)
        k = vertex % 3
        cut = np.empty((3, 3))
        cut[k] = [*rng.uniform(-0.15, 0.15, 2), 0.0]
        cut[(k + 1) % 3] = [*rng.uniform(-0.9, 0.9, 2), rng.uniform(0.5, 1.0)]
        cut[(k + 2) % 3] = [*rng.uniform(-0.9, 0.9, 2), -rng.uniform(0.5, 1.0)]
        shift = rng.uniform(-0.3, 0.3, 3)
        base, cut = (base + shift) @ q.T, (cut + shift) @ q.T
        cut[k] += lift * U * rng.choice([-1.0, 1.0]) * q[:, 2] * rng.integers(1, 4)
        pair = np.concatenate([cut, base] if vertex < 3 else [base, cut])
        if _uncertain(*base, cut[k]) and oracle.pair(pair)["T"] > 1e-4:
            out.append(pair)
    return np.array(out)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("lift", [0.0, 0.25, 1.0])
@pytest.mark.parametrize("vertex", range(6))
def test_one_vertex_near_the_plane(vertex, lift, precision):
    import parity_checks as pc
    import torch

    from paper_2606_06511_amd import ttie

    n = 40
    x = _pairs_near(vertex, lift, n, 10 * vertex + int(4 * lift)).reshape(-1, 3)
    tris = np.arange(6 * n, dtype=np.int32).reshape(2 * n, 3)
    pairs = np.arange(2 * n, dtype=np.int32).reshape(n, 2)
    ref = pc.reference(x, tris, pairs)
    assert len(ref["hit_pair"]) == n
    ctx = ttie.Context(0)
    ctx.reserve(len(x), len(tris), n, max_hits=n, max_blocks=36 * n)
    out = ctx.evaluate(*[torch.from_numpy(a).cuda() for a in (x, tris, pairs)], precision=precision, flags=True, pair_T=True)
    ctx.check()
    pc.check_eval_outputs(out, ref, pairs, tris, precision)
    pc.check_hits(ctx.hits(), ref, pairs, precision)
