"""Resident launches that are given up (their workgroups were not all resident):
the call goes on from the state the launch began with, launch by launch for
int16 weights, with the sweeps for real-valued ones."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_1104_3830_amd as sk  # noqa: E402
import skgen  # noqa: E402

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]

BUDGET = 2048  # iterations of one resident launch


@pytest.fixture(scope="module")
def ctx():
    c = sk.Context(0, arena_bytes=256 << 20)
    yield c
    c.close()


def give_up(ctx, launch, workgroup, polls=0):
    f = sk.lib().sk_test_resident_give_up
    f.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    f.restype = None
    f(ctx._ptr, launch, workgroup, polls)


@pytest.mark.parametrize("polls", [0, 200])
@pytest.mark.parametrize("launch,workgroup", [(0, 0), (0, 5), (1, 9)])
@pytest.mark.parametrize("n", [300, 1000])
def test_int16_goes_on_bitwise(ctx, n, launch, workgroup, polls):
    W = torch.from_numpy(skgen.uniform_weights(n, 0, 100, seed=n)).cuda()
    prm = sk.make_params([1, 2], tol=0.0, max_iters=1501)
    want = ctx.scale(W, prm)
    give_up(ctx, launch, workgroup, polls)
    got = ctx.scale(W, prm)
    assert got.report["iters_stage"] == want.report["iters_stage"]
    assert torch.equal(got.potentials, want.potentials)


@pytest.mark.parametrize("polls", [0, 200])
@pytest.mark.parametrize("n,ladder,tol", [(300, [1000, 200, 1000], 3e-3), (700, [400, 100, 400], 3e-3),
                                          (700, [400, 100, 400], 3e-4)])
def test_real_goes_on_from_an_odd_iteration(ctx, n, ladder, tol, polls):
    """The first launch ends where stage 1 has converged, at an odd iteration;
    the second finds that, runs stage 2 and is dropped at its end. The sweeps
    then find stage 1 converged as well, without another iteration."""
    W = torch.from_numpy(skgen.euclidean_real(n, seed=n)).cuda()
    cap = 1501
    for _ in range(12):
        prm = sk.make_params(ladder, tol=tol, max_iters=cap)
        want = ctx.scale_real(W, prm)
        stages = want.report["iters_stage"][:3]
        assert stages[0] == cap and stages[1] < cap
        if cap + stages[1] == BUDGET:
            break
        cap = BUDGET - stages[1]
    assert cap + stages[1] == BUDGET and stages[1] % 2 == 1
    give_up(ctx, 1, 3, polls)
    got = ctx.scale_real(W, prm)
    assert got.report["iters_stage"][:2] == stages[:2]
    # stage 2 by the sweeps: its FP32 sums may pass the tolerance a few
    # iterations earlier or later
    assert abs(got.report["iters_stage"][2] - stages[2]) <= 0.02 * stages[2] + 1
    if got.report["stages_capped"] == 1:
        assert got.report["residual_fp64"] <= 1.02 * tol
    assert np.isfinite(got.report["ub"])
