"""Real-valued log-weights at the sizes of the resident iteration (n <= 1024),
at the edges of its blocks (32 rows) and chunks (512 columns), against the
FP64 oracle. Tolerances as in test_gpu_real: 1e-4 on log x for entries >= 1e-6
after a fixed number of iterations."""
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


def weights(n, kind):
    W = skgen.euclidean_real(n, seed=n)
    if kind == "sparse":
        off = (np.arange(n * n).reshape(n, n) * 2654435761 >> 7) % 2 == 0
        np.fill_diagonal(off, False)
        W[off] = -np.inf
    return W


def check(W, p, pot, ub, vb):
    B = W.astype(np.float64) - float(W.max())
    lu, lv = sk.split_potentials(pot, W.shape[0])
    fin = np.isfinite(B)
    Lg = np.where(fin, p * np.where(fin, B, 0) + lu[:, None] + lv[None, :], -np.inf)
    Lo = np.where(fin, p * (np.where(fin, B, 0) + ub[:, None] + vb[None, :]), -np.inf)
    sig = Lo > np.log(1e-6)
    assert sig.any() and np.abs(Lg[sig] - Lo[sig]).max() < 1e-4


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 255, 511, 512, 513, 1000, 1023, 1024, 1025])
@pytest.mark.parametrize("kind", ["dense", "sparse"])
def test_fixed_iterations_match_oracle(ctx, n, kind):
    W = weights(n, kind)
    ladder, it = [20, 60], 9
    res = ctx.scale_real(dev(W), sk.make_params(ladder, tol=0.0, max_iters=it))
    assert res.report["iters_stage"][:2] == [it, it]
    B = W.astype(np.float64) - float(W.max())
    ub, vb = np.zeros(n), np.zeros(n)
    for p in ladder:
        ub, vb, _, _ = oracle.sinkhorn(B, p, 0.0, it, ub, vb)
    check(W, ladder[-1], res.potentials, ub, vb)


@pytest.mark.parametrize("n", [50, 700])
def test_sums_outside_the_safe_range(ctx, n):
    """A column far below every row maximum (left to the sweeps) and a start
    at zero potentials with p w down to -1400 (row sums underflow)."""
    W = weights(n, "dense") * 7.0
    W[:, 3] -= 60.0
    p, B = 100, W.astype(np.float64) - float(W.max())
    pot = torch.zeros(sk.potentials_bytes(n), dtype=torch.uint8, device="cuda")
    for warm in (False, True):
        res = ctx.scale_real(dev(W), sk.make_params([p], tol=0.0, max_iters=4, warm_start=warm),
                             potentials=pot.clone())
        ub, vb, _, _ = oracle.sinkhorn(B, p, 0.0, 4)
        check(W, p, res.potentials, ub, vb)


@pytest.mark.parametrize("n", [40, 600])
def test_empty_row_or_column(ctx, n):
    for cut in (np.s_[n // 2, :], np.s_[:, n // 2]):
        W = weights(n, "dense")
        W[cut] = -np.inf
        with pytest.raises(sk.SkError) as e:
            ctx.scale_real(dev(W), sk.make_params([20], tol=1e-4, max_iters=20))
        assert e.value.status == sk.SK_ENOSUPPORT
