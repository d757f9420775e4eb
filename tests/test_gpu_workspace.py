"""The workspace's broad-phase regions: their size, and the leaf region lent to the spring pattern,
filled to its last entry."""

import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _bytes(ctx, tris):
    from paper_2606_06511_amd import ttie

    n = ctypes.c_size_t()
    lim = ttie.Limits(16, tris, 16, 16, 16)
    assert ttie.lib().ttie_workspace_size(ctx.handle, ctypes.byref(lim), ctypes.byref(n)) == ttie.TTIE_OK
    return n.value


def test_bytes_of_a_triangle():
    """Sort 16, tree boxes 64, leaves 24, float64 box and centre 60, hash entries 8 x 28 (the room for
    handed-over work no longer grows at these sizes)."""
    from paper_2606_06511_amd import ttie

    ctx = ttie.Context(0)
    n = 1 << 20
    assert _bytes(ctx, 3 * n) - _bytes(ctx, 2 * n) <= n * (16 + 64 + 24 + 60 + 8 * 28) + 4096


@pytest.mark.parametrize("n", [1, 2, 43, 1000])
def test_spring_pattern_fills_the_leaf_region(n):
    """Triangles without a common vertex list 6 neighbours each, the most; the next regions hold what
    a broad phase before and after finds."""
    import torch

    from paper_2606_06511_amd import ttie

    x = torch.from_numpy(np.random.default_rng(n).normal(size=(3 * n, 3))).cuda()
    tris = torch.arange(3 * n, dtype=torch.int32, device="cuda").reshape(n, 3)
    ctx = ttie.Context(0)
    ctx.reserve(3 * n, n, n * n, max_hits=16)

    def pairs():
        p, k = ctx.broadphase(x, tris)
        ctx.check()
        p = p[: int(k.item())].long()
        return torch.sort(p[:, 0] * n + p[:, 1]).values

    before = pairs()
    row_ptr, col = ctx.springs_pattern(tris, 3 * n)
    want = 3 * (torch.arange(3 * n, device="cuda") // 3)[:, None] + torch.arange(3, device="cuda")
    assert torch.equal(row_ptr.long(), 3 * torch.arange(3 * n + 1, device="cuda"))
    assert torch.equal(col.long().reshape(-1, 3), want)
    assert torch.equal(pairs(), before)
