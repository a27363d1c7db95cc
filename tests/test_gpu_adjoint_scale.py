"""Mixed adjoint solves whose loss gradient is far from 1: an FP32 solve of H
lambda = dL is homogeneous, so a scaled dL gives the scaled lambda, or, where
FP32 squares no longer hold the scale, a solve reported as not converged --
never a zero reported as the solution.  Scales within FP32's squares must
solve: those of the preconditioned vector M^-1 r, whose largest entry can be
|r| over the preconditioner's least constant, a thousandth of the mean Hessian
diagonal.  The norm of the right-hand side is a sum in FP64 at any scale.
Tolerances: lambda to the solve's rtol 1e-6 times the condition of these coarse
grids' preconditioned system (below 1e2), the norm to FP32's rounding of each
entry (2^-24)."""
import numpy as np
import pytest

from paper_0911_1407_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", params=[(32, 32, 32), (16, 24, 256)], ids=["plane", "passes"])
def solved(request):
    from paper_0911_1407_amd import binding
    n = request.param
    inst = synth.make_instance(n, tuple(8.0 * v for v in n), 1.2, 1.1, 1.3, radius=4.0 * n[0], mask_frac=0.2, seed=5,
                               block=4)
    plan = binding.Plan(n, inst["box"], precision="mixed")
    plan.set_instance(inst)
    s = inst["s_true"]
    dL = np.random.default_rng(8).standard_normal(n)
    out, info = plan.adjoint(s, dL, rtol=1e-6, max_cg=500)
    assert info["status"] == 0
    d = inst["beta"] ** 2 * inst["nbar"] * inst["w"] * np.exp(inst["beta"] * s)
    top = np.abs(np.fft.rfftn(dL)).max() / (1e-3 * d.mean())  # bound of |M^-1 r|
    return plan, s, dL, out["lam"].cpu().numpy(), info["grad0"], top


@pytest.mark.parametrize("scale", [1e-15, 1e12, 1e-30, 1e20, 1e30])
def test_scaled_loss_gradient(solved, scale):
    from paper_0911_1407_amd import binding
    plan, s, dL, lam, bnorm, top = solved
    out, info = plan.adjoint(s, scale * dL, rtol=1e-6, max_cg=500)
    assert abs(info["grad0"] - scale * bnorm) <= 1e-6 * scale * bnorm, info
    got = out["lam"].cpu().numpy() / scale
    if scale > 1e-16 and (scale * top) ** 2 < 1e38:
        assert info["status"] == 0, info
    if info["status"] == 0:
        assert np.linalg.norm(got - lam) <= 1e-4 * np.linalg.norm(lam), info
    else:
        assert info["status"] == binding.PL_ERR_NOT_CONVERGED and info["rel_grad"] > 1e-6, info


@pytest.mark.parametrize("precision", [0, 1])
def test_a_right_hand_side_beyond_the_vectors_range(solved, precision):
    # 1e45 is beyond FP32, within FP64
    from paper_0911_1407_amd import binding
    plan, s, dL, lam, bnorm, top = solved
    out, info = plan.adjoint(s, 1e45 * dL, rtol=1e-6, max_cg=500, precision=precision)
    if precision == 0:
        assert info["status"] == 0
        assert np.linalg.norm(out["lam"].cpu().numpy() / 1e45 - lam) <= 1e-4 * np.linalg.norm(lam)
    else:
        assert info["status"] == binding.PL_ERR_NOT_CONVERGED and not info["rel_grad"] <= 1e-6, info
    # without a value there is nothing to solve
    with pytest.raises(binding.PLError) as e:
        plan.adjoint(s, np.nan * dL, rtol=1e-6, max_cg=500, precision=precision)
    assert e.value.code == binding.PL_ERR_DOMAIN
