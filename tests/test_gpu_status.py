"""The latched status: returned once, to the context that latched it, on any stream and from any
thread."""

import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side_stream", [False, True])
@pytest.mark.parametrize("n_ctx", [1, 2, 5])
def test_returned_once(n_ctx, side_stream):
    import torch

    from paper_2606_06511_amd import ttie

    x = torch.from_numpy(np.random.default_rng(0).normal(size=(6, 3))).cuda()
    tris = torch.tensor([[0, 1, 2], [3, 4, 5]], dtype=torch.int32, device="cuda")
    good = torch.tensor([[0, 1]], dtype=torch.int32, device="cuda")
    bad = torch.tensor([[0, 7]], dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    seen, errors = {}, []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream() if side_stream else torch.cuda.current_stream()):
                ctx = ttie.Context(0)
                ctx.reserve(6, 2, 4, max_hits=4)
                got = []
                for it in range(20):
                    ctx.evaluate(x, tris, bad if (it + k) % 2 else good)
                    got += [ctx.status(), ctx.status()]
                seen[k] = got
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(n_ctx)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    for k, got in seen.items():
        want = []
        for it in range(20):
            want += [ttie.TTIE_ERR_INDEX_OUT_OF_RANGE if (it + k) % 2 else ttie.TTIE_OK, ttie.TTIE_OK]
        assert got == want
