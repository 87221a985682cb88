"""A potential has one form, log = k + f, however long it stays on chip: row
sums whose logarithm is next to a half integer, where k + f and (k + 1) +
(f - 1) are a rounding apart. The bits depend neither on how a run is split
into launches or calls nor on what it runs beside."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_1104_3830_amd as sk  # noqa: E402
import skgen  # noqa: E402

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]


@pytest.fixture(scope="module")
def ctx():
    c = sk.Context(0)
    yield c
    c.close()


def start_near_half(n):
    """Starting potentials with log v_j = G_j + gam_j, gam_j within 1e-4 of
    +-1/2 and |G_j| <= 40; on a diagonal matrix of zeros row j's sum is v_j."""
    rng = np.random.default_rng(n)
    G = rng.integers(-40, 41, n).astype(np.int32)
    gam = (rng.choice([-1.0, 1.0], n) * (0.5 - 1e-4 * rng.random(n) ** 2)).astype(np.float32)
    z = np.zeros(n, np.int32)
    raw = np.concatenate([z.view(np.uint8), np.zeros(n, np.float32).view(np.uint8), G.view(np.uint8),
                          gam.view(np.uint8)])
    return torch.from_numpy(raw).cuda(), G.astype(np.float64) + gam.astype(np.float64)


def diagonal(n, real):
    W = np.full((n, n), -np.inf, np.float32) if real else np.full((n, n), sk.SENTINEL, np.int16)
    np.fill_diagonal(W, 0)
    return torch.from_numpy(W).cuda()


def run(ctx, W, iters, pot):
    prm = sk.make_params([1], tol=0.0, max_iters=iters, warm_start=True)
    f = ctx.scale_real if W.dtype == torch.float32 else ctx.scale
    return f(W, prm, potentials=pot.clone()).potentials


@pytest.mark.parametrize("real", [False, True])
@pytest.mark.parametrize("n", [64, 128, 192, 256, 300, 512, 513, 1024])
def test_fractions_next_to_one_half(ctx, n, real):
    W, (pot, lv) = diagonal(n, real), start_near_half(n)
    got = run(ctx, W, 1, pot)
    raw = got.cpu().numpy().view(np.float32).reshape(4, n)
    lu, _ = sk.split_potentials(got, n)
    # the logarithm of a float32 sum, and its rounding to a fraction
    assert np.abs(lu + lv).max() <= 4 * 2.0 ** -24
    assert np.abs(raw[1]).max() <= 0.5001 and np.abs(raw[3]).max() <= 0.5001
    # two iterations in one call, and in two
    assert torch.equal(run(ctx, W, 2, pot), run(ctx, W, 1, got))
    if not real:
        prm = sk.make_params([1], tol=0.0, max_iters=2, warm_start=True)
        other = torch.from_numpy(skgen.uniform_weights(300, 0, 50, seed=1)).cuda()
        z = ctx.new_potentials(300)
        whole = run(ctx, W, 2, pot)
        few = ctx.scale_batch([W, other], prm, potentials=[pot.clone(), z.clone()])
        many = ctx.scale_batch([other] * 33 + [W], prm, potentials=[z.clone() for _ in range(33)] + [pot.clone()])
        assert torch.equal(few[0].potentials, whole) and torch.equal(many[-1].potentials, whole)
