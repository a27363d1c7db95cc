"""The largest planes, whose grids take plane passes or separate ones by the number
of planes, the operation and the precision: operators on both sides of each line,
against the oracle.  Tolerances as for the other plane grids: FFT roundoff times
the spread of 1/lambda, 1e-11 relative in FP64 and 2e-5 in FP32."""
import numpy as np
import pytest

from conftest import assert_elementwise, oracle_problem
from oracle import model as o_model
from oracle import newton as o_newton
from paper_0911_1407_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GRIDS = [
    (24, 128, 128), (32, 128, 128),                    # gradient
    (12, 256, 64), (32, 256, 64), (64, 256, 64), (96, 256, 64),  # FP64: whole, half, gradient; FP32: half
    (32, 64, 192), (48, 64, 192), (96, 64, 192), (48, 192, 64), (48, 256, 48),
    (48, 96, 192), (64, 96, 192), (96, 96, 192),       # the largest FP64 planes of 192 points
    (32, 192, 96), (48, 192, 96), (32, 96, 256), (48, 96, 256), (96, 128, 192),  # FP32 only from here
    (48, 256, 128), (96, 256, 128), (48, 192, 192), (64, 192, 192), (128, 192, 192),
]


@pytest.mark.parametrize("n", GRIDS)
def test_operators_match_oracle(n):
    from paper_0911_1407_amd import binding
    inst = synth.make_instance(n, tuple(8.0 * v for v in n), 1.2, 1.1, 1.3, radius=4.0 * max(n), mask_frac=0.2, seed=3,
                               block=2)
    P = oracle_problem(inst)
    rng = np.random.default_rng(6)
    s = inst["s_true"] + 0.05 * rng.standard_normal(n)
    v = rng.standard_normal(n)
    plan = binding.Plan(n, inst["box"], precision="mixed")
    plan.set_instance(inst)
    g, _ = plan.grad(s)
    g_ref, hv_ref = o_model.gradient(P, s), o_model.hessvec(P, s, v)
    assert np.linalg.norm(g.cpu().numpy() - g_ref) <= 1e-11 * np.linalg.norm(g_ref)
    assert_elementwise(g.cpu().numpy(), g_ref, 1e-10, what=f"gradient {n}")
    hv = plan.hessvec(v).cpu().numpy()
    assert np.linalg.norm(hv - hv_ref) <= 1e-11 * np.linalg.norm(hv_ref)
    assert_elementwise(hv, hv_ref, 1e-10, what=f"HVP {n}")
    v32 = torch.from_numpy(v).cuda().float()
    hv32 = torch.empty_like(v32)
    binding.pl_hessvec_f32(plan.h, None, v32, hv32)
    assert np.linalg.norm(hv32.double().cpu().numpy() - hv_ref) <= 2e-5 * np.linalg.norm(hv_ref)
    v_hat = np.fft.rfftn(v)
    ref = o_newton.SpectralOps(P).hessvec(o_model.hess_diag(P, s), v_hat)
    vt = torch.from_numpy(v_hat).cuda()
    for dtype, tol in ((torch.complex128, 1e-11), (torch.complex64, 2e-5)):
        out = plan.hessvec_hat(vt.to(dtype)).cpu().numpy()
        assert np.linalg.norm(out - ref) <= tol * np.linalg.norm(ref), dtype
