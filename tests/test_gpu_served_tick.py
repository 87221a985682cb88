"""The served loop at its shortest tick: requests of every size class move."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_1104_3830_amd as sk  # noqa: E402
import skgen  # noqa: E402

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]


@pytest.mark.parametrize("n", [200, 300, 700, 1100])
def test_one_iteration_per_tick(monkeypatch, n):
    monkeypatch.setenv("SK_SERVE_ITERS_PER_TICK", "1")
    W, sigma = skgen.planted(n, seed=n)
    ctx = sk.Context(0)
    try:
        ticket = ctx.submit(W, sk.make_params([1, 2, 4], tol=1e-5, max_iters=50, threshold=1e-4))
        end = time.time() + 20
        got = None
        while got is None and time.time() < end:
            got = ctx.poll(ticket, n)
            time.sleep(0.001)
        assert got is not None, "the request did not finish"
        st, perm, weight, rep = got
        assert st == sk.SK_OK and weight == 1050 * n and np.array_equal(perm, sigma)
    finally:
        ctx.close()
