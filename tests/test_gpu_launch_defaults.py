"""Launch parameters at their defaults: setting what ttie_get_param reports changes no launch, the
autotuner's choices hold the defaults, and lists on both sides of the length at which the screening's
split changes, whatever the buffer is reserved for."""

import json

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _launches(torch, path, run):
    """The (kernel, grid) of everything that run launches (three times, lest a record is dropped)."""
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        for _ in range(3):
            run()
        torch.cuda.synchronize()
    prof.export_chrome_trace(str(path))
    events = json.loads(path.read_text())["traceEvents"]
    return {(e["name"], tuple(e["args"]["grid"])) for e in events if "grid" in e.get("args", {})}


def test_reported_values_are_the_defaults(tmp_path):
    import torch

    from paper_2606_06511_amd import autotune, ttie, workloads

    x, tris = workloads.folded_cloth(2, n=64)
    xd, td = torch.from_numpy(x).cuda(), torch.from_numpy(tris).cuda()
    ctx = ttie.Context(0)
    ctx.reserve(len(x), len(tris), 1 << 21, max_hits=1 << 12)
    pairs, n = ctx.broadphase(xd, td)
    ctx.evaluate(xd, td, pairs, n)
    ctx.check()

    def run():
        ctx.evaluate(xd, td, pairs, n)
        ctx.bsr_symbolic(len(x))

    default = _launches(torch, tmp_path / "a.json", run)
    if not default:
        pytest.skip("no kernel records in this environment")
    for name, (pid, values) in autotune.SPACE.items():
        assert ctx.get_param(pid) in values, name
    for p in range(5):
        ctx.set_param(p, ctx.get_param(p))
    assert _launches(torch, tmp_path / "b.json", run) == default
    ctx.set_param(ttie.PARAM_SCREEN_BLOCKS, 64)
    assert ("k_screen", 64) in [(k.split("(")[0].split("::")[-1], g[0]) for k, g in _launches(torch, tmp_path / "c.json", run)]


@pytest.mark.parametrize("blocks", [0, 64, 2000, 65536])
@pytest.mark.parametrize("n", [1, 65, 64 * 6144 - 1, 1 << 22, (1 << 22) + 1, 64 * 12288 * 6 + 63])
def test_lists_in_a_large_buffer(n, blocks):
    """The split follows the list's length, not the buffer's: a short list in a large buffer, and both
    sides of 2^22 candidates."""
    import torch

    from paper_2606_06511_amd import ttie, workloads

    x, tris = workloads.folded_cloth(2, n=64)
    pairs = oracle.pairs(x, tris).astype(np.int32)
    ref = oracle.evaluate(x, tris, pairs, hessian=False)["flags"]
    take = torch.from_numpy(np.random.default_rng(n).integers(0, len(pairs), n)).cuda()
    want = torch.from_numpy(ref).cuda()[take]
    cap = max(n, 5_000_000)
    buf = torch.zeros((cap, 2), dtype=torch.int32, device="cuda")
    buf[:n] = torch.from_numpy(pairs).cuda()[take]
    hits = int((want == 1).sum().item())
    ctx = ttie.Context(0)
    ctx.reserve(len(x), len(tris), cap, max_hits=max(64, hits), max_blocks=64)
    ctx.set_param(ttie.PARAM_SCREEN_BLOCKS, blocks)
    out = ctx.evaluate(torch.from_numpy(x).cuda(), torch.from_numpy(tris).cuda(), buf,
                       torch.tensor([n], device="cuda"), hessian=False, flags=True)
    ctx.check()
    assert torch.equal(out["flags"][:n], want)
    assert int(out["n_hits"].item()) == hits


def test_a_set_budget_is_taken_as_it_is():
    """Half of the default budget is what a mesh of few groups takes by itself: set, it hands over as
    many batches of candidates (the workspace's tenth word; 3 % is several times what the arbitrary
    order inside the sort's buckets changes), and the whole default fewer."""
    import torch

    from paper_2606_06511_amd import ttie

    rng = np.random.default_rng(0)
    n = 300_000
    x = torch.from_numpy((rng.uniform(0.0, 42.0, (n, 1, 3)) + rng.normal(0.0, 0.4, (n, 3, 3))).reshape(-1, 3)).cuda()
    tris = torch.arange(3 * n, dtype=torch.int32, device="cuda").reshape(n, 3)
    ctx = ttie.Context(0)
    ctx.reserve(3 * n, n, 8_000_000, max_hits=64)
    head = -ctx.workspace.data_ptr() % 256

    def batches(value):
        ctx.set_param(ttie.PARAM_TRAV_BUDGET, value)
        total = 0
        for _ in range(4):
            ctx.broadphase(x, tris)
            ctx.check()
            total += ctx.workspace[head : head + 40].view(torch.int32)[9].item()
        return total

    default = batches(0)
    assert default > 1000
    assert abs(batches(64) - default) <= 0.03 * default
    assert batches(128) < 0.97 * default
