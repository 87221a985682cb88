"""Stored K with one iteration per stage: that iteration is the log-domain one
before K is formed, so the result is that of the sweeps over int16 W."""
import pytest

torch = pytest.importorskip("torch")
import paper_1104_3830_amd as sk  # noqa: E402
import skgen  # noqa: E402

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]


@pytest.mark.parametrize("n", [1, 15, 513, 1100])
@pytest.mark.parametrize("storage", ["bf16", "f32"])
@pytest.mark.parametrize("ladder", [[3], [1, 2, 4]])
def test_one_iteration_per_stage(n, storage, ladder):
    W = torch.from_numpy(skgen.uniform_weights(n, 0, 60, seed=n)).cuda()
    ctx = sk.Context(0, arena_bytes=64 << 20)
    ctx.arena.fill_(0xFF)  # NaN wherever nothing was written
    got = ctx.scale(W, sk.make_params(ladder, tol=0.0, max_iters=1, storage=storage))
    a, b = sk.split_potentials(got.potentials, n)
    ref = ctx.scale(W, sk.make_params(ladder, tol=0.0, max_iters=1))
    c, d = sk.split_potentials(ref.potentials, n)
    # a step per stage, FP32 sums of n terms in chains of at most 64, doubled
    # by each of the two stage changes
    tol = 14 * 64 * 2.0 ** -24
    assert abs(a - c).max() <= tol and abs(b - d).max() <= tol
    for key in ("residual_fp64", "col_residual_fp64", "ub"):
        assert abs(got.report[key] - ref.report[key]) <= 1e-4 * (1 + abs(ref.report[key]))
