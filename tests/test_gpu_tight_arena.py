"""Arenas of every size around what a call needs: one that is large enough stays
large enough when it grows, also by so much that the resident iteration's
exchange area fits but not what is taken beside it; the results are the same,
and nothing is written behind the arena."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_1104_3830_amd as sk  # noqa: E402
import skgen  # noqa: E402
from tests.tight import TightContext  # noqa: E402

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]


def sweep(sizes, call):
    """call(ctx) over the sizes: the results of those from the first that
    suffices on."""
    got = []
    for nbytes in sizes:
        ctx = TightContext(0, arena_bytes=nbytes)
        try:
            got.append(call(ctx))
            torch.cuda.synchronize()
        except sk.SkError as e:
            assert e.status == sk.SK_ENOMEM and not got, (nbytes, str(e))
        assert ctx.guard_untouched(), nbytes
        ctx.close()
    assert len(got) > 1
    return got


@pytest.mark.parametrize("n", [300, 304])
def test_scale(n):
    W = torch.from_numpy(skgen.uniform_weights(n, 0, 100, seed=n)).cuda()
    prm = sk.make_params([1, 2], tol=0.0, max_iters=20)
    full = sk.lib().sk_arena_bytes(n, 0)
    got = sweep(range(full // 8, full + 2048, 2048), lambda ctx: ctx.scale(W, prm).potentials)
    # the smallest have room for the sweeps alone, whose sums are of another
    # order; from the middle kernels' room on the bits are the same, with the
    # exchange area or without
    first = [torch.equal(g, got[-1]) for g in got].index(True)
    assert all(torch.equal(g, got[-1]) for g in got[first:])
    want = np.concatenate(sk.split_potentials(got[-1], n))
    for g in got[:first]:
        assert np.abs(np.concatenate(sk.split_potentials(g, n)) - want).max() < 1e-4


@pytest.mark.parametrize("option", [{}, {"storage": "bf16"}, {"method": "newton"}])
def test_solve(option):
    n = 300
    W = torch.from_numpy(skgen.planted(n, seed=n)[0]).cuda()
    # several evaluated stages, the reduced matrix shrinking from one to the next
    prm = sk.make_params([1, 2, 4], tol=1e-6, max_iters=50, threshold=1e-30, opt_ratio=1.0, **option)
    full = sk.lib().sk_solve_arena_bytes(n, prm.storage, n * n)
    got = sweep(range(full // 8, full, 8192), lambda ctx: ctx.solve(W, prm))
    for g in got:
        # the sweeps' sums, in the smallest arenas, are of another order
        assert g["weight"] == 1050 * n and g["nnz"] == got[-1]["nnz"]
        a, b = (np.concatenate(sk.split_potentials(r["potentials"], n)) for r in (g, got[-1]))
        assert np.abs(a - b).max() < 1e-4


def test_solve_real():
    n = 300
    W = torch.from_numpy(skgen.euclidean_real(n, seed=1)).cuda()
    prm = sk.paper_params(n, ladder=[100, 150, 200, 250])
    full = sk.lib().sk_real_arena_bytes(n, n * n // 4)
    got = sweep(range(full // 8, full, 8192), lambda ctx: ctx.solve_real(W, prm))
    for g in got:
        assert g["status"] == got[-1]["status"] and g["weight"] == pytest.approx(got[-1]["weight"], rel=1e-12)
        assert np.array_equal(g["perm"], got[-1]["perm"])
