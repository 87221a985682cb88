"""Served requests that ask for the single pass: the serving thread sweeps every
instance in two passes, and they give what the others give."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_1104_3830_amd as sk  # noqa: E402
import skgen  # noqa: E402

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]


@pytest.mark.parametrize("n", [64, 512, 1200])
def test_single_pass_request_is_served(n):
    W, sigma = skgen.planted(n, seed=n)
    results = []
    for fused in (False, True):
        ctx = sk.Context(0)
        try:
            prm = sk.make_params([1, 2, 4], tol=1e-5, max_iters=50, threshold=1e-4, fused=fused)
            ticket = ctx.submit(W, prm)
            end, got = time.time() + 20, None
            while got is None and time.time() < end:
                got = ctx.poll(ticket, n)
                time.sleep(0.001)
            assert got is not None
            results.append(got)
        finally:
            ctx.close()
    (st0, perm0, weight0, rep0), (st1, perm1, weight1, rep1) = results
    assert st0 == st1 == sk.SK_OK and weight0 == weight1 == 1050 * n
    assert np.array_equal(perm0, perm1) and np.array_equal(perm0, sigma)
    assert rep0["iters_stage"] == rep1["iters_stage"] and rep0["residual_fp64"] == rep1["residual_fp64"]
