"""Contexts that come and go while a stream is captured in the default (global) error mode, on the
capturing thread and on another: the capture stays valid, and creating and destroying succeed."""

import ctypes
import threading

import pytest

pytestmark = pytest.mark.gpu


def _create(ttie):
    h = ctypes.c_void_p()
    return ttie.lib().ttie_create(0, ctypes.byref(h)), h


@pytest.mark.parametrize("other_thread", [False, True])
def test_contexts_during_a_capture(other_thread):
    import torch

    from paper_2606_06511_amd import ttie, workloads

    x, tris = workloads.folded_cloth(2, n=48)
    xd, td = torch.from_numpy(x).cuda(), torch.from_numpy(tris).cuda()
    ctx = ttie.Context(0)
    ctx.reserve(len(x), len(tris), 1 << 16, max_hits=1 << 12)
    pairs, n = ctx.broadphase(xd, td)
    out = ctx.evaluate(xd, td, pairs, n)
    ctx.check()
    want = out["energy"].item()
    assert want > 0.0
    st, before = _create(ttie)
    assert st == ttie.TTIE_OK
    torch.cuda.synchronize()
    seen = []

    def come_and_go():
        seen.append(ttie.lib().ttie_destroy(before))
        st, h = _create(ttie)
        seen.append(st)
        seen.append(ttie.lib().ttie_destroy(h) if st == ttie.TTIE_OK else None)

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.broadphase(xd, td, out=(pairs, n))
        if other_thread:
            t = threading.Thread(target=come_and_go)
            t.start()
            t.join()
        else:
            come_and_go()
        ctx.evaluate(xd, td, pairs, n, out=out)
    assert seen == [ttie.TTIE_OK] * 3
    for _ in range(3):
        out["energy"].zero_()
        g.replay()
        torch.cuda.synchronize()
        assert out["energy"].item() == want
        ctx.check()
