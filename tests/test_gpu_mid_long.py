"""Thousands of iterations in a batch (a launch each) and alone (resident): a
fraction that rounding takes past 1/2 is moved to its integer part in both, so
the potentials stay bitwise equal. Such roundings are rare (some in 1e7); these
instances meet them."""
import pytest

torch = pytest.importorskip("torch")
import paper_1104_3830_amd as sk  # noqa: E402
import skgen  # noqa: E402

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]


def test_long_runs_in_a_batch_and_alone():
    cases = [(327, 543), (569, 507), (668, 559), (893, 609), (928, 607)]
    Ws = [torch.from_numpy(skgen.uniform_weights(n, 0, 1000, seed=s)).cuda() for n, s in cases]
    prm = sk.make_params([1, 2, 4, 8, 16, 32], tol=1e-5, max_iters=500)
    ctx = sk.Context(0)
    for W, b in zip(Ws, ctx.scale_batch(Ws, prm)):
        a = ctx.scale(W, prm)
        assert a.report["iters_total"] == b.report["iters_total"] > 2500
        assert torch.equal(a.potentials, b.potentials)
