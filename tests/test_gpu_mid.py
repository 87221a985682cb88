"""Instances iterated by one launch per iteration (256 < n <= 1024), at the
edges of its row blocks (32 rows) and column chunks (512 columns), against the
FP64 oracle. Tolerances as in test_gpu_parity (1e-4 on log x for entries
>= 1e-6 after a fixed number of iterations)."""
import numpy as np
import pytest

import oracle
import paper_1104_3830_amd as sk
import skgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


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


@pytest.mark.parametrize("n", [257, 288, 289, 511, 512, 513, 520, 777, 1000, 1023, 1024, 1025])
@pytest.mark.parametrize("sparse", [False, True])
def test_fixed_iterations_match_oracle(ctx, n, sparse):
    """Three stages of 7 iterations (an odd count: a stage ends on either
    launch of a pair); sparse: half of the entries absent."""
    W = skgen.uniform_weights(n, 0, 60, seed=n)
    if sparse:
        off = (np.arange(n * n).reshape(n, n) * 2654435761 >> 7) % 2 == 0
        np.fill_diagonal(off, False)
        W[off] = sk.SENTINEL
    ladder, it = [1, 3, 4], 7
    res = ctx.scale(dev(W), sk.make_params(ladder, tol=0.0, max_iters=it))
    assert res.report["iters_stage"][:3] == [it] * 3 and res.report["stages_capped"] == 3
    B = oracle.log_weights(W)
    ub, vb = np.zeros(n), np.zeros(n)
    for p in ladder:
        ub, vb, _, _ = oracle.sinkhorn(B, p, 0.0, it, ub, vb)
    assert_same_x(W, ladder[-1], res.potentials, ub, vb)


def test_unaligned_base(ctx):
    """n a multiple of 8 with a base that is not 16-byte aligned (scalar
    loads): bitwise the aligned matrix's result."""
    n = 400
    W = dev(skgen.uniform_weights(n, 0, 100, seed=3))
    flat = torch.zeros(n * n + 8, dtype=torch.int16, device="cuda")
    V = flat[1:1 + n * n].view(n, n)
    V.copy_(W)
    prm = sk.make_params([1, 2], tol=0.0, max_iters=9)
    assert V.data_ptr() % 16 != 0
    assert torch.equal(ctx.scale(V, prm).potentials, ctx.scale(W, prm).potentials)


@pytest.mark.parametrize("n", [300, 1001])
def test_sums_outside_the_safe_range(ctx, n):
    """Column 7 far below every row maximum and a start at zero potentials
    (every row sum overflows): both take the exact max shift."""
    W = skgen.uniform_weights(n, 0, 1000, seed=n)
    W[:, 7] = (W[:, 7] // 10).astype(np.int16)
    p, B = 4, oracle.log_weights(W)
    pot = torch.zeros(sk.potentials_bytes(n), dtype=torch.uint8, device="cuda")
    for warm in (False, True):
        res = ctx.scale(dev(W), sk.make_params([p], tol=0.0, max_iters=3, warm_start=warm),
                        potentials=pot.clone())
        ub, vb, _, _ = oracle.sinkhorn(B, p, 0.0, 3)
        assert_same_x(W, p, res.potentials, ub, vb)


@pytest.mark.parametrize("n", [40, 300, 700])
def test_starting_potentials_in_any_split(ctx, n):
    """log u = F + phi and log v = G + gam given with the whole value in the
    float part (not a fraction): the same iterate, up to the float32 rounding
    of the given values (2^-20 at |log| <= 16)."""
    W = skgen.uniform_weights(n, 0, 10, seed=n)
    rng = np.random.default_rng(n)
    lv = rng.uniform(-9, 9, n).astype(np.float32).astype(np.float64)
    split = torch.from_numpy(sk.pack_potentials(np.zeros(n), lv)).cuda()
    z = np.zeros(n, np.int32)
    raw = np.concatenate([z.view(np.uint8), np.zeros(n, np.float32).view(np.uint8), z.view(np.uint8),
                          lv.astype(np.float32).view(np.uint8)])
    prm = sk.make_params([2], tol=0.0, max_iters=3, warm_start=True)
    a = ctx.scale(dev(W), prm, potentials=split)
    b = ctx.scale(dev(W), prm, potentials=torch.from_numpy(raw).cuda())
    for x, y in zip(sk.split_potentials(a.potentials, n), sk.split_potentials(b.potentials, n)):
        assert np.abs(x - y).max() < 1e-5


@pytest.mark.parametrize("n", [300, 600])
def test_stage_counts_and_convergence(ctx, n):
    """A planted instance converges at the oracle's iterations in every stage
    and its whole solve finds the planted optimum."""
    W, sigma = skgen.planted(n, seed=n)
    out = ctx.solve(dev(W), sk.make_params([1, 2, 4], tol=1e-5, max_iters=50, threshold=1e-4, opt_ratio=1.5))
    assert out["weight"] == 1050 * n and np.array_equal(out["perm"], sigma)
    out = ctx.solve(dev(W), sk.make_params([1, 2, 4], tol=1e-5, max_iters=50, threshold=1e-4))
    assert out["report"]["iters_stage"][:3] == [1, 1, 1] and out["report"]["optimal_proved"] == 1


@pytest.mark.parametrize("n", [300, 900])
def test_empty_row_or_column(ctx, n):
    for cut in (np.s_[n // 2, :], np.s_[:, n // 2]):
        W = skgen.uniform_weights(n, 0, 10, seed=1)
        W[cut] = sk.SENTINEL
        with pytest.raises(sk.SkError) as e:
            ctx.scale(dev(W), sk.make_params([1, 2], tol=1e-6, max_iters=50))
        assert e.value.status == sk.SK_ENOSUPPORT


@pytest.mark.parametrize("n", [257, 300, 512, 513, 800, 1023, 1024])
@pytest.mark.parametrize("tol,cap", [(0.0, 11), (1e-4, 400)])
def test_resident_and_launched_iterations_agree_bitwise(ctx, n, tol, cap):
    """One instance iterates in a resident launch, a batch with a launch per
    iteration; few instances take the column step in the same launch, many in
    one of its own: the same bits, iterations and residuals either way."""
    W = skgen.uniform_weights(n, 0, 50, seed=n)
    W[n // 3, n // 5:] = sk.SENTINEL
    prm = sk.make_params([1, 2, 3], tol=tol, max_iters=cap)
    Wd = dev(W)
    one = ctx.scale(Wd, prm)
    few = ctx.scale_batch([Wd, dev(skgen.uniform_weights(280, 0, 50, seed=1))], prm)[0]
    many = ctx.scale_batch([Wd] + [dev(skgen.uniform_weights(1000 - k, 0, 50, seed=k)) for k in range(9)], prm)[0]
    for other in (few, many):
        assert one.report["iters_stage"] == other.report["iters_stage"]
        assert one.report["residual_fp32"] == other.report["residual_fp32"]
        assert torch.equal(one.potentials, other.potentials)


def test_resident_run_longer_than_a_launch(ctx):
    """More iterations than one resident launch takes."""
    W = dev(skgen.uniform_weights(270, 0, 100, seed=4))
    prm = sk.make_params([2], tol=0.0, max_iters=4200)
    one = ctx.scale(W, prm)
    assert one.report["iters_total"] == 4200
    two = ctx.scale_batch([W, W], prm)
    assert torch.equal(one.potentials, two[0].potentials) and torch.equal(one.potentials, two[1].potentials)
