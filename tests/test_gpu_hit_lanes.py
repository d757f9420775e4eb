"""The derivatives of a hit come from two lanes, one per end of the interval: hit counts around a
wave's 32 hits, and every kind of end, against the oracle, at the bars of tests/parity_checks.py."""

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
