"""The solvers' products: matrices whose columns name rows without blocks (a pattern that is not
symmetric: such a column multiplies zeros), and the matrix-free and coupled rows around the kernels'
splits (64 rows a block, 256 a partial, eight incidences a turn), against dense solves."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _one_sided(seed, n):
    """Diagonally dominant symmetric blocks on two thirds of the rows; every such row also holds
    blocks in columns of the others, whose rows are empty."""
    rng = np.random.default_rng(seed)
    live = np.sort(rng.choice(n, max(1, 2 * n // 3), replace=False))
    dead = np.setdiff1d(np.arange(n), live)
    blocks = {(int(r), int(r)): np.zeros((3, 3)) for r in live}
    for r in live:
        for c in rng.choice(live, min(len(live), 4), replace=False):
            if r != c:
                v = rng.normal(size=(3, 3))
                blocks[int(r), int(c)], blocks[int(c), int(r)] = v, v.T
    scale = max([sum(np.abs(b).sum(1).max() for (r, _), b in blocks.items() if r == q) for q in live] + [1.0])
    for r in live:
        blocks[int(r), int(r)] = 2.0 * scale * np.eye(3)
        for c in rng.choice(dead, min(len(dead), int(rng.integers(1, 12))), replace=False) if len(dead) else ():
            blocks[int(r), int(c)] = 1e3 * scale * rng.normal(size=(3, 3))
    keys = sorted(blocks)
    ptr = np.searchsorted([r for r, _ in keys], np.arange(n + 1)).astype(np.int32)
    col = np.array([c for _, c in keys], np.int32)
    vals = np.array([blocks[k] for k in keys])
    b = rng.normal(size=(n, 3))
    b[dead] = 0.0
    return ptr, col, vals, b, np.repeat(np.isin(np.arange(n), live), 3)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [2, 3, 64, 97, 400])
def test_columns_without_a_row(n, precision):
    import torch

    from paper_2606_06511_amd import ttie

    ptr, col, vals, b, keep = _one_sided(n, n)
    dense = oracle.bsr_to_dense(ptr, col, vals, n)
    dt = torch.float64 if precision == "fp64" else torch.float32
    ctx = ttie.Context(0)
    ctx.reserve(n, 1, 16, max_hits=16)
    # condition number at most 3 (eigenvalues within [0.5, 1.5] of the diagonal's scale); float32
    # vectors round at 6e-8
    tol, bar = (1e-12, 1e-11) if precision == "fp64" else (1e-6, 1e-5)
    up = [torch.from_numpy(ptr).cuda(), torch.from_numpy(col).cuda(), torch.from_numpy(vals).cuda().to(dt)]
    want = np.zeros(3 * n)
    want[keep] = np.linalg.solve(dense[np.ix_(keep, keep)], b.reshape(-1)[keep])
    # a solve over every row first: its vectors are what the next ones find in the workspace
    eye = torch.eye(3, dtype=dt, device="cuda").repeat(n, 1, 1)
    every = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    for s in (1.0, -2.0):
        ctx.pcg(every, every[:n].clone(), 1e3 * eye, torch.rand((n, 3), dtype=dt, device="cuda"), max_iter=1, tol=0.0)
        x, info = ctx.pcg(*up, torch.from_numpy(b).cuda().to(dt), scale=s, mu_rel=0.0, max_iter=200, tol=tol)
        ctx.check()
        got = x.double().cpu().numpy().reshape(-1)
        assert np.array_equal(got[~keep], np.zeros((~keep).sum()))
        assert np.linalg.norm(got - s * want) <= bar * np.linalg.norm(s * want)
        assert 0 < info[0].item() < 200


def _crossed(n, extra=0):
    """One triangle crossed by n others: 3 n + 3 rows, three of them with n incidences; `extra`
    vertices of no triangle."""
    rng = np.random.default_rng(n)
    k = np.arange(n)
    at = np.stack([0.5 + k % 16, 0.5 + k // 16, 0.0 * k], 1)[:, None, :]
    small = at + np.array([[-0.2, 0.1, -0.3], [0.25, 0.05, -0.2], [0.0, -0.1, 0.4]]) + rng.uniform(-0.05, 0.05, (n, 3, 3))
    x = np.concatenate([np.array([[-5.0, -5.0, 0.01], [60.0, -4.0, -0.02], [-4.0, 60.0, 0.015]]), small.reshape(-1, 3)])
    tris = np.arange(3 * (n + 1), dtype=np.int32).reshape(-1, 3)
    pairs = np.stack([np.zeros(n, np.int32), k + 1], 1).astype(np.int32)
    return np.concatenate([x, 100.0 + np.arange(3.0 * extra).reshape(extra, 3)]), tris, pairs


def _evaluated(n, precision, extra=0):
    import torch

    from paper_2606_06511_amd import ttie

    x, tris, pairs = _crossed(n, extra)
    ctx = ttie.Context(0)
    ctx.reserve(len(x), len(tris), n, max_hits=n, max_blocks=36 * n)
    out = ctx.evaluate(*[torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (x, tris, pairs)], precision=precision)
    ctx.check()
    assert int(out["n_hits"].item()) == n
    nb, nv = int(out["n_blocks"].item()), len(x)
    ptr, col = out["row_ptr"].cpu().numpy(), out["col_idx"][:nb].cpu().numpy()
    val = out["vals"][:nb].double().cpu().numpy()
    return ctx, out, oracle.bsr_to_dense(ptr, col, val, nv)


# rows: 6, 9, 24, 27, 63, 66, 255, 258, 603; incidences of the long ones: 1 to 200
SIZES = [1, 2, 7, 8, 9, 20, 21, 84, 85, 200]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n", SIZES)
def test_matrix_free_rows(n, precision):
    ctx, out, H = _evaluated(n, precision)
    # |x - x*| <= |A^-1| (|b - A x|), the true residual within tol + 8 roundings an iteration of the
    # recursion's
    tol, u = (1e-12, 2.0**-53) if precision == 0 else (1e-6, 2.0**-24)
    d, info = ctx.pcg_mf(out["grad"], scale=-1.0, mu_rel=1.0, max_iter=400, tol=tol)
    ctx.check()
    it, _, mu, _ = info.cpu().numpy()
    A = H + mu * np.eye(len(H))
    g = out["grad"].double().cpu().numpy().reshape(-1)
    want = np.linalg.solve(A, -g)
    got = d.double().cpu().numpy().reshape(-1)
    assert 0 < it < 400
    assert np.linalg.norm(got - want) <= np.linalg.cond(A) * (tol + 8 * (it + 1) * u) * np.linalg.norm(want)


@pytest.mark.parametrize("n", SIZES)
def test_coupled_rows(n):
    """K on some rows only (the hits' other rows are still solved for), vertices of neither."""
    import torch

    ctx, out, H = _evaluated(n, 0, extra=5)
    nv = len(H) // 3
    rng = np.random.default_rng(n)
    rows = np.sort(rng.choice(nv - 2, (nv - 2) // 2, replace=False))  # the last two vertices are in neither
    R = rng.normal(size=(3 * len(rows), 3 * len(rows)))
    keepb = np.triu(rng.random((len(rows), len(rows))) < min(1.0, 8.0 / len(rows)), 1)
    keepb = keepb | keepb.T
    D = np.where(np.kron(keepb, np.ones((3, 3))) > 0, R + R.T, 0.0)
    D += (1.0 + np.abs(D).sum(1).max()) * np.eye(len(D))
    at = -np.ones(nv, int)
    at[rows] = np.arange(len(rows))
    hold = [[c for c in range(nv) if at[c] >= 0 and (c == r or keepb[at[r], at[c]])] if at[r] >= 0 else [] for r in range(nv)]
    ptr = np.cumsum([0] + [len(h) for h in hold]).astype(np.int32)
    col = np.array([c for h in hold for c in h], np.int32)
    val = np.array([D[3 * at[r] : 3 * at[r] + 3, 3 * at[c] : 3 * at[c] + 3] for r in range(nv) for c in hold[r]])
    K = oracle.bsr_to_dense(ptr, col, val, nv)
    w = np.trace(D) / max(np.trace(H), 1e-300)
    mu, tol = float(np.trace(D)) / len(D), 1e-12
    b = rng.normal(size=(nv, 3))
    b[nv - 2 :] = 0.0
    live = (np.abs(K) + np.abs(H)).reshape(nv, 3, -1).sum((1, 2)) > 0
    b[~live] = 0.0
    up = [torch.from_numpy(np.asarray(a)).cuda() for a in (ptr, col, val)]
    d, info = ctx.pcg_coupled(*up, w, torch.from_numpy(b).cuda(), scale=1.0, mu=mu, max_iter=400, tol=tol)
    ctx.check()
    it = info[0].item()
    A = K + w * H + mu * np.eye(len(H))
    want = np.linalg.solve(A, b.reshape(-1))
    got = d.cpu().numpy().reshape(-1)
    assert 0 < it < 400
    assert np.array_equal(got.reshape(nv, 3)[~live], np.zeros(((~live).sum(), 3)))
    assert np.linalg.norm(got - want) <= np.linalg.cond(A) * (tol + 8 * (it + 1) * 2.0**-53) * np.linalg.norm(want)
