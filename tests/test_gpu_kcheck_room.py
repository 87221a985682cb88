"""The FP64 check of a stored K under a tile table of 16-row segments: it stays
inside an arena of the stated size, and finds what it finds with the shipped
table."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_1104_3830_amd as sk  # noqa: E402
import skgen  # noqa: E402
from tests.tight import TightContext  # noqa: E402

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]


@pytest.mark.parametrize("n", [512, 1000, 2048])
@pytest.mark.parametrize("storage", [1, 2])
def test_stored_k_check_with_16_row_segments(n, storage):
    W = torch.from_numpy(skgen.uniform_weights(n, 0, 100, seed=n)).cuda()
    prm = sk.make_params([1, 2], tol=0.0, max_iters=4, storage=storage)
    want = sk.Context(0).scale(W, prm)
    table = list(sk.loaded_tile_table)
    try:
        sk.set_tile_table([(65536, 16)])
        ctx = TightContext(0, arena_bytes=sk.lib().sk_arena_bytes(n, storage))
        got = ctx.scale(W, prm)
        torch.cuda.synchronize()
        assert ctx.guard_untouched()
    finally:
        sk.set_tile_table(table)
    # column sums in another order: eight steps of FP32 sums of n terms in
    # chains of at most 64, and an entry of K may round to its neighbour
    tol = 8 * 64 * 2.0 ** -24 + (2.0 ** -8 if storage == 1 else 2.0 ** -23)
    for key in ("residual_fp64", "col_residual_fp64"):
        assert abs(got.report[key] - want.report[key]) <= tol * (1 + want.report[key])
    assert np.isfinite(got.report["ub"])
