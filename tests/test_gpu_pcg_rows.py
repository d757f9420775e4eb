"""PCG over ragged block rows: row counts around the kernels' splits (64 rows a block, 256 a
partial), rows of 0 to 40 blocks (eight lanes share a row), rows without blocks."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _matrix(seed, n, longest):
    """A symmetric block matrix with ragged rows, diagonally dominant by a factor of two (eigenvalues
    within [0.5, 1.5] of the diagonal's scale), some rows without any block."""
    rng = np.random.default_rng(seed)
    empty = set(rng.choice(n, n // 5, replace=False).tolist()) if n >= 5 else set()
    live = [r for r in range(n) if r not in empty]
    blocks = {}
    for r in live:
        for c in rng.choice(live, min(len(live), int(rng.integers(0, longest // 2 + 1))), replace=False):
            if r != c:
                v = rng.normal(size=(3, 3))
                blocks[r, int(c)] = v
                blocks[int(c), r] = v.T
    rows = {r: sorted([c for (a, c) in blocks if a == r] + [r]) for r in live}
    scale = max([sum(np.abs(blocks[r, c]).sum(1).max() for c in rows[r] if c != r) for r in live] + [1.0])
    ptr, col, vals = [0], [], []
    for r in range(n):
        for c in rows.get(r, []):
            col.append(c)
            vals.append(2.0 * scale * np.eye(3) if c == r else blocks[r, c])
        ptr.append(len(col))
    dense = np.zeros((3 * n, 3 * n))
    for r in range(n):
        for k in range(ptr[r], ptr[r + 1]):
            dense[3 * r : 3 * r + 3, 3 * col[k] : 3 * col[k] + 3] = vals[k]
    b = rng.normal(size=(n, 3))
    b[sorted(empty)] = 0.0
    return np.array(ptr, np.int32), np.array(col, np.int32), np.array(vals), dense, b


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,longest", [(1, 2), (2, 2), (63, 6), (64, 12), (65, 40), (255, 6), (256, 6), (257, 20), (700, 10)])
def test_pcg_ragged_rows(n, longest, precision):
    import torch

    from paper_2606_06511_amd import ttie

    ptr, col, vals, dense, b = _matrix(n, n, longest)
    dt = torch.float64 if precision == "fp64" else torch.float32
    dev = torch.device("cuda", 0)
    ctx = ttie.Context(0)
    ctx.reserve(n, 1, 16, max_hits=16)
    # the residual bound times the condition number (at most 3): 3e-12; float32 vectors round at 6e-8
    tol, bar = (1e-12, 1e-11) if precision == "fp64" else (1e-6, 1e-5)
    x, info = ctx.pcg(torch.from_numpy(ptr).to(dev), torch.from_numpy(col).to(dev),
                      torch.from_numpy(vals).to(dev, dt).contiguous(), torch.from_numpy(b).to(dev, dt).contiguous(),
                      scale=-1.0, mu_rel=0.0, max_iter=200, tol=tol)
    ctx.check()
    live = np.diff(ptr) > 0
    keep = np.repeat(live, 3)
    want = np.zeros(3 * n)
    want[keep] = np.linalg.solve(dense[np.ix_(keep, keep)], -b.reshape(-1)[keep])
    got = x.double().cpu().numpy().reshape(-1)
    assert np.array_equal(got[~keep], np.zeros((~keep).sum()))
    assert np.linalg.norm(got - want) <= bar * max(np.linalg.norm(want), 1e-300)
    it, resid, _, xb = info.cpu().numpy()
    assert 0 < it < 200 and resid <= tol
    assert abs(xb - got @ -b.reshape(-1)) <= 1e-6 * abs(xb)
