"""The derivatives of a hit come from two lanes, one per end of the interval: hit counts around a
wave's 32 hits, and every kind of end; and rows of the assembly around the lengths that its kernels read at once; against
the oracle, at the bars of tests/parity_checks.py."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 65, 129])
def test_counts_around_a_wave(n, precision):
    import parity_checks as pc
    import torch

    from paper_2606_06511_amd import ttie

    rng = np.random.default_rng(n)
    x, k = [], 0
    while k < n:  # crossing pairs, apart from each other, in every order of their vertices
        p = rng.normal(size=(2, 3, 3))
        if oracle.pair(p.reshape(6, 3))["T"] > 0.0:
            x.append(p.reshape(6, 3) + np.array([20.0 * k, 0.0, 0.0]))
            k += 1
    x = np.concatenate(x)
    tris = np.arange(6 * n, dtype=np.int32).reshape(2 * n, 3)
    pairs = np.arange(2 * n, dtype=np.int32).reshape(n, 2)
    ref = pc.reference(x, tris, pairs)
    assert len(ref["hit_pair"]) == n
    ctx = ttie.Context(0)
    ctx.reserve(len(x), len(tris), n, max_hits=n, max_blocks=36 * n)
    dev = [torch.from_numpy(a).cuda() for a in (x, tris, pairs)]
    out = ctx.evaluate(*dev, precision=precision, flags=True, pair_T=True)
    ctx.check()
    pc.check_eval_outputs(out, ref, pairs, tris, precision)
    pc.check_hits(ctx.hits(), ref, pairs, precision)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 6, 11, 12, 13, 24, 25, 47, 100])
def test_rows_of_many_hits(n, precision):
    """One triangle crossed by n others, so that its three rows hold n incidences each and 6 n
    column candidates of 3 n + 3 columns."""
    import parity_checks as pc
    import torch

    from paper_2606_06511_amd import ttie

    rng = np.random.default_rng(n)
    k = np.arange(n)
    at = np.stack([0.5 + k % 10, 0.5 + k // 10, 0.0 * k], 1)[:, None, :]
    small = at + np.array([[-0.2, 0.1, -0.3], [0.25, 0.05, -0.2], [0.0, -0.1, 0.4]]) + rng.uniform(-0.05, 0.05, (n, 3, 3))
    x = np.concatenate([np.array([[-5.0, -5.0, 0.01], [40.0, -4.0, -0.02], [-4.0, 40.0, 0.015]]), small.reshape(-1, 3)])
    tris = np.arange(3 * (n + 1), dtype=np.int32).reshape(-1, 3)
    pairs = np.stack([np.zeros(n, np.int32), k + 1], 1).astype(np.int32)[rng.permutation(n)]
    ref = pc.reference(x, tris, pairs)
    assert len(ref["hit_pair"]) == n
    ctx = ttie.Context(0)
    ctx.reserve(len(x), len(tris), n, max_hits=n, max_blocks=36 * n)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (x, tris, pairs)]
    out = ctx.evaluate(*dev, precision=precision, flags=True, pair_T=True)
    ctx.check()
    pc.check_eval_outputs(out, ref, pairs, tris, precision)
