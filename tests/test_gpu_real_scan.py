"""The range scan of real-valued weights reads every entry once, whatever the
alignment of W: extremes, NaN and +inf at the ends of the array are seen."""
import pytest

torch = pytest.importorskip("torch")
import paper_1104_3830_amd as sk  # noqa: E402

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]


@pytest.mark.parametrize("n", [2, 5, 63, 260, 515])
@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_scan_sees_both_ends(n, offset):
    ctx = sk.Context(0)
    prm = sk.make_params([1], tol=0.0, max_iters=1, prescale=True)
    buf = torch.full((n * n + offset,), -1.0, device="cuda")
    W = buf[offset:].view(n, n)
    for lo, hi in ((0, n * n - 1), (n * n - 1, 0)):
        W.fill_(-1.0)
        W.view(-1)[lo] = -8.0
        W.view(-1)[hi] = 0.0
        # the range 8 is a power of two: its reciprocal is exact
        assert ctx.scale_real(W, prm).report["p_scale"] == 0.125
    for at in (0, n * n - 1):
        for bad in (float("nan"), float("inf")):
            W.fill_(-1.0)
            W.view(-1)[at] = bad
            with pytest.raises(sk.SkError) as e:
                ctx.scale_real(W, prm)
            assert e.value.status == sk.SK_EINVAL
