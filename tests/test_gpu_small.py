"""Instances small enough for the one-workgroup kernel (n <= 256), at the
edges of its size classes (64 columns per class, 16 rows per wave), against
the FP64 oracle. Tolerances as in test_gpu_parity: 1e-4 on log x for entries
>= 1e-6 after a fixed number of iterations (its terms come from the same
table, and it adds them in FP64 across lanes)."""
import numpy as np
import pytest

import oracle
import paper_1104_3830_amd as sk
import skgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EDGES = [1, 2, 3, 15, 17, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257]


@pytest.fixture(scope="module")
def ctx():
    c = sk.Context(0)
    yield c
    c.close()


def dev(W):
    return torch.from_numpy(np.ascontiguousarray(W)).cuda()


def assert_same_x(W, p, pot, ub_o, vb_o):
    B = oracle.log_weights(W)
    lu, lv = sk.split_potentials(pot, W.shape[0])
    with np.errstate(invalid="ignore"):
        Lg = p * B + lu[:, None] + lv[None, :]
        Lo = p * (B + ub_o[:, None] + vb_o[None, :])
    sig = Lo > np.log(1e-6)
    assert sig.any()
    assert np.abs(Lg - Lo)[sig].max() < 1e-4


@pytest.mark.parametrize("n", EDGES)
@pytest.mark.parametrize("sparse", [False, True])
def test_fixed_iterations_match_oracle(ctx, n, sparse):
    """Three stages of 12 iterations; sparse: half of the entries absent (the
    diagonal kept), so that rows and columns mix absent and present ones."""
    W = skgen.uniform_weights(n, 0, 60, seed=n)
    if sparse:
        off = (np.arange(n * n).reshape(n, n) * 2654435761 >> 7) % 2 == 0
        np.fill_diagonal(off, False)
        W[off] = sk.SENTINEL
    ladder, it = [1, 3, 4], 12
    res = ctx.scale(dev(W), sk.make_params(ladder, tol=0.0, max_iters=it))
    assert res.report["iters_stage"][:3] == [it] * 3 and res.report["stages_capped"] == 3
    B = oracle.log_weights(W)
    ub, vb = np.zeros(n), np.zeros(n)
    for p in ladder:
        ub, vb, _, _ = oracle.sinkhorn(B, p, 0.0, it, ub, vb)
    assert_same_x(W, ladder[-1], res.potentials, ub, vb)


@pytest.mark.parametrize("n", [40, 100, 160, 250])
def test_sums_outside_the_safe_range(ctx, n):
    """Column 7 far below every row maximum (its sum underflows at the first
    iteration) and a start at zero potentials, where every row sum overflows:
    both are recomputed with the exact max shift."""
    W = skgen.uniform_weights(n, 0, 1000, seed=n)
    W[:, 7] = (W[:, 7] // 10).astype(np.int16)
    p, B = 4, oracle.log_weights(W)
    pot = torch.zeros(sk.potentials_bytes(n), dtype=torch.uint8, device="cuda")
    for warm in (False, True):
        res = ctx.scale(dev(W), sk.make_params([p], tol=0.0, max_iters=3, warm_start=warm),
                        potentials=pot.clone())
        ub, vb, _, _ = oracle.sinkhorn(B, p, 0.0, 3)
        assert_same_x(W, p, res.potentials, ub, vb)


@pytest.mark.parametrize("n", [50, 120, 180, 230])
def test_long_stage_over_several_launches_is_bitwise(ctx, n):
    """5000 iterations of one stage (several launches of the kernel) equal
    1700 and 3300 resumed, and the same instance within a mixed batch."""
    W = dev(skgen.uniform_weights(n, 0, 100, seed=n))

    def prm(iters, warm=False):
        return sk.make_params([2], tol=0.0, max_iters=iters, warm_start=warm)

    whole = ctx.scale(W, prm(5000))
    first = ctx.scale(W, prm(1700))
    rest = ctx.scale(W, prm(3300, True), potentials=first.potentials.clone())
    assert whole.report["iters_total"] == 5000
    assert torch.equal(whole.potentials, rest.potentials)
    others = [dev(skgen.uniform_weights(m, 0, 100, seed=m)) for m in (30, 70, 150, 300, 256)]
    mixed = ctx.scale_batch(others[:2] + [W] + others[2:], prm(5000))
    assert torch.equal(whole.potentials, mixed[2].potentials)


@pytest.mark.parametrize("n", [20, 70, 140, 200])
def test_empty_row_or_column(ctx, n):
    for cut in (np.s_[n // 2, :], np.s_[:, n // 2]):
        W = skgen.uniform_weights(n, 0, 10, seed=1)
        W[cut] = sk.SENTINEL
        with pytest.raises(sk.SkError) as e:
            ctx.scale(dev(W), sk.make_params([1, 2], tol=1e-6, max_iters=50))
        assert e.value.status == sk.SK_ENOSUPPORT
