"""The finalise of the column step over its forms: more row segments than a
thread holds in registers, capped stages (the last workgroup moves what the
others wrote), several instances, and columns at the edge of a group of 64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_1104_3830_amd as sk  # noqa: E402
import skgen  # noqa: E402

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]


def logs(res, n):
    return np.concatenate(sk.split_potentials(res.potentials, n))


@pytest.mark.parametrize("n", [4160, 4200])
def test_more_segments_than_slots(n):
    # segments of 16 rows: 260 and 263 column slots
    W = torch.from_numpy(skgen.uniform_weights(n, 0, 1000, seed=3)).cuda()
    prm = sk.make_params([1, 2], tol=0.0, max_iters=3)
    ctx = sk.Context(0)
    want = logs(ctx.scale(W, prm), n)
    table = list(sk.loaded_tile_table)
    try:
        sk.set_tile_table([(65536, 16)])
        got = logs(ctx.scale(W, prm), n)
    finally:
        sk.set_tile_table(table)
    # six steps, each within 2 * 16 FP32 roundings of a sum's two orders
    assert np.abs(got - want).max() <= 6 * 32 * 2.0 ** -24


@pytest.mark.parametrize("n", [1025, 1088, 1100, 2047])
def test_capped_stages_and_batches(n):
    # one iteration per stage, every stage capped: the stage change reads the
    # column potentials of the same launch
    W = torch.from_numpy(skgen.uniform_weights(n, 0, 400, seed=n)).cuda()
    prm = sk.make_params([1, 2, 4], tol=0.0, max_iters=1)
    ctx = sk.Context(0)
    a = ctx.scale(W, prm)
    assert a.report["iters_total"] == 3 and a.report["stages_capped"] == 3
    lu, lv = np.zeros(n), np.zeros(n)
    w = W.cpu().numpy().astype(np.float64)
    lu = -w.max(1)

    def lse(x, axis):
        m = x.max(axis, keepdims=True)
        return np.squeeze(m, axis) + np.log(np.exp(x - m).sum(axis))

    for s, p in enumerate((1, 2, 4)):
        if s:
            lu, lv = 2 * lu, 2 * lv
        lu = -lse(p * w + lv[None, :], 1)
        lv = -lse(p * w + lu[:, None], 0)
    # FP32 sums of n terms in trees and chains of at most 64, twice a stage,
    # doubled by each stage change
    assert np.abs(logs(a, n) - np.concatenate((lu, lv))).max() <= 14 * 64 * 2.0 ** -24
    b = ctx.scale_batch([W, W[: n - 1, : n - 1].contiguous()], prm)
    assert np.array_equal(logs(b[0], n), logs(a, n))
