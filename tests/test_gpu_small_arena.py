"""Arenas that hold what the sweeps need and not what the middle kernels and the
batched check take beside it: every call runs, and gives the result of a roomy
arena (the same bits, except where the sweeps take sizes of the middle
kernels). The sizes are those that the sizing functions gave before these
kernels were there."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_1104_3830_amd as sk  # noqa: E402
import skgen  # noqa: E402
from tests.tight import TightContext  # noqa: E402

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]


def uniform(n, seed):
    return torch.from_numpy(skgen.uniform_weights(n, 0, 60, seed=seed)).cuda()


def logs(pot, n):
    return np.concatenate(sk.split_potentials(pot, n))


def same(a, b, n, bits):
    assert a.report["iters_stage"] == b.report["iters_stage"]
    if bits:
        assert torch.equal(a.potentials, b.potentials)
    # seven steps of FP32 sums in chains of at most 64 terms, doubled once
    assert np.abs(logs(a.potentials, n) - logs(b.potentials, n)).max() <= 14 * 64 * 2.0 ** -24
    for key in ("residual_exact_fp64", "col_residual_exact_fp64", "ub"):
        x, y = a.report[key], b.report[key]
        assert abs(x - y) <= 1e-4 * (1 + abs(y)), key


@pytest.mark.parametrize("count,n,nbytes", [(64, 1024, 4065280), (64, 1000, 4047360), (64, 300, 13375488),
                                            (512, 1, 7247360), (64, 64, 901120), (64, 256, 1433600),
                                            (4, 2048, 3665152)])
def test_batches(count, n, nbytes):
    Ws = [uniform(n, k) for k in range(count)]
    prm = sk.make_params([1, 2], tol=0.0, max_iters=4)
    roomy = sk.Context(0).scale_batch(Ws, prm)
    ctx = TightContext(0, arena_bytes=nbytes)
    tight = ctx.scale_batch(Ws, prm)
    assert ctx.guard_untouched()
    for a, b in zip(tight, roomy):
        same(a, b, n, bits=not 256 < n <= 1024)


@pytest.mark.parametrize("n,storage,nbytes", [(1024, 0, 137472), (300, 0, 235776), (256, 0, 44288), (1000, 1, 3241472),
                                              (1000, 2, 5241344), (2048, 0, 1758976)])
def test_one_instance(n, storage, nbytes):
    W = uniform(n, n)
    prm = sk.make_params([1, 2], tol=0.0, max_iters=4, storage=storage)
    roomy = sk.Context(0).scale(W, prm)
    ctx = TightContext(0, arena_bytes=nbytes)
    tight = ctx.scale(W, prm)
    assert ctx.guard_untouched()
    same(tight, roomy, n, bits=storage or not 256 < n <= 1024)


@pytest.mark.parametrize("n,nbytes", [(1, 29696), (64, 31744), (300, 61184), (1000, 152576), (1024, 154112)])
def test_real(n, nbytes):
    W = torch.from_numpy(skgen.euclidean_real(n, seed=n)).cuda()
    prm = sk.make_params([20, 40], tol=0.0, max_iters=4)
    roomy = sk.Context(0).scale_real(W, prm)
    ctx = TightContext(0, arena_bytes=nbytes)
    tight = ctx.scale_real(W, prm)
    assert ctx.guard_untouched()
    same(tight, roomy, n, bits=False)


@pytest.mark.parametrize("ns", [[1000], [300, 1000, 64], [777] * 40, [1001, 2000]])
def test_the_stated_size_holds_the_fastest_plan(ns):
    """In an arena of exactly the size that the sizing functions give, the bits
    are those of a roomy one."""
    import ctypes
    Ws = [uniform(n, k) for k, n in enumerate(ns)]
    prm = sk.make_params([1, 2], tol=0.0, max_iters=4)
    size = sk.lib().sk_batch_arena_bytes(len(ns), (ctypes.c_int32 * len(ns))(*ns), 0)
    ctx, roomy = TightContext(0, arena_bytes=size), sk.Context(0, arena_bytes=256 << 20)
    for a, b, n in zip(ctx.scale_batch(Ws, prm), roomy.scale_batch(Ws, prm), ns):
        same(a, b, n, bits=True)
    assert ctx.guard_untouched()
    if len(ns) == 1:
        X = torch.from_numpy(skgen.euclidean_real(ns[0], seed=1)).cuda()
        ctx = TightContext(0, arena_bytes=sk.lib().sk_real_arena_bytes(ns[0], 0))
        same(ctx.scale_real(X, prm), roomy.scale_real(X, prm), ns[0], bits=True)
        assert ctx.guard_untouched()


def test_a_smaller_plan_is_no_error():
    ctx = TightContext(0, arena_bytes=154112)
    prm = sk.make_params([1], tol=1e-1, max_iters=400)
    ctx.scale(uniform(1024, 1), prm)
    assert ctx.last_error() == ""
    ctx.scale_real(torch.from_numpy(skgen.euclidean_real(1024, seed=1)).cuda(), prm)
    assert ctx.last_error() == ""


def test_served():
    """A served request whose region only has the sweeps' room."""
    n = 1024
    W, sigma = skgen.planted(n, seed=1)
    ctx = TightContext(0, arena_bytes=int((2 * n * n + 160000) * 4 / 3) + 4096)
    try:
        ticket = ctx.submit(W, sk.make_params([1, 2, 4], tol=1e-5, max_iters=50, threshold=1e-4))
        end, got = time.time() + 20, None
        while got is None and time.time() < end:
            got = ctx.poll(ticket, n)
            time.sleep(0.001)
        assert got is not None
        assert got[0] == sk.SK_OK and got[2] == 1050 * n and np.array_equal(got[1], sigma)
        assert ctx.guard_untouched()
    finally:
        ctx.close()
