"""Starting potentials whose integer parts need more than the 28 bits in which
the resident iteration exchanges G: adding c to every log v and taking it from
every log u moves nothing else."""
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


def start(n, c):
    raw = np.zeros((4, n), np.int32)
    raw[0] = -c
    raw[2] = c
    return torch.from_numpy(raw.view(np.uint8).reshape(-1)).cuda()


def parts(pot, n):
    raw = pot.cpu().numpy().view(np.int32).reshape(4, n)
    return raw[0].astype(np.int64), raw[1].view(np.float32), raw[2].astype(np.int64), raw[3].view(np.float32)


@pytest.mark.parametrize("c", [3 << 26, 3 << 25, -(3 << 26), (1 << 27) - 1, 1 - (1 << 27)])
@pytest.mark.parametrize("n", [64, 300, 1000])
def test_int16_one_stage(ctx, n, c):
    """Exponents are integer sums, in which c cancels: the same bits."""
    W = torch.from_numpy(skgen.uniform_weights(n, 0, 40, seed=n)).cuda()
    prm = sk.make_params([2], tol=0.0, max_iters=3, warm_start=True)
    F0, p0, G0, g0 = parts(ctx.scale(W, prm, potentials=start(n, 0)).potentials, n)
    F1, p1, G1, g1 = parts(ctx.scale(W, prm, potentials=start(n, c)).potentials, n)
    assert np.array_equal(F1, F0 - c) and np.array_equal(G1, G0 + c)
    assert np.array_equal(p0, p1) and np.array_equal(g0, g1)


# past 28 bits from the second stage on, where p doubles (4 G stays within the
# 2^30 of the padding columns' exponent)
@pytest.mark.parametrize("c", [3 << 25, -(3 << 25), (1 << 27) - 9])
@pytest.mark.parametrize("n", [64, 300, 1000])
def test_int16_two_stages(ctx, n, c):
    W = torch.from_numpy(skgen.uniform_weights(n, 0, 40, seed=n)).cuda()
    prm = sk.make_params([1, 2], tol=0.0, max_iters=3, warm_start=True)
    F0, p0, G0, g0 = parts(ctx.scale(W, prm, potentials=start(n, 0)).potentials, n)
    F1, p1, G1, g1 = parts(ctx.scale(W, prm, potentials=start(n, c)).potentials, n)
    # the stage change scales in FP64, where a logarithm of size 2^29 has 2^-24
    # left; then six steps of FP32 sums in chains of at most 64 terms
    tol = 2.0 ** -24 + 6 * 64 * 2.0 ** -24
    assert np.abs((F1 + 2 * c - F0) + (p1.astype(np.float64) - p0)).max() <= tol
    assert np.abs((G1 - 2 * c - G0) + (g1.astype(np.float64) - g0)).max() <= tol


@pytest.mark.parametrize("c", [3 << 26, 3 << 25, -(3 << 26), (1 << 27) - 1])
@pytest.mark.parametrize("n", [64, 300, 1000])
def test_real(ctx, n, c):
    W = torch.from_numpy(skgen.euclidean_real(n, seed=n)).cuda()
    prm = sk.make_params([20, 40], tol=0.0, max_iters=3, warm_start=True)
    F0, p0, G0, g0 = parts(ctx.scale_real(W, prm, potentials=start(n, 0)).potentials, n)
    F1, p1, G1, g1 = parts(ctx.scale_real(W, prm, potentials=start(n, c)).potentials, n)
    # six steps of FP32 sums in chains of at most 64 terms, doubled by the
    # stage change, and exponents of size 2^29 in FP64, twice a step
    tol = 12 * 64 * 2.0 ** -24 + 12 * 2.0 ** (29 - 52)
    assert np.abs((F1 + 2 * c - F0) + (p1.astype(np.float64) - p0)).max() <= tol
    assert np.abs((G1 - 2 * c - G0) + (g1.astype(np.float64) - g0)).max() <= tol
