"""Plane passes (y and z transforms of an x plane in one launch) against the
oracle, at the sizes where they can go wrong: every transform length on both
axes, planes whose columns or row pairs do not fill a wave, the largest planes
that fit a workgroup's LDS, and the first ones that do not (which take the
separate passes).  Tolerances are those of the operators: FFT roundoff times
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
    (8, 8, 8), (8, 12, 16), (12, 16, 12),   # transforms of one thread each
    (8, 32, 48), (8, 48, 32), (8, 64, 96),  # short lengths, ragged last waves
    (8, 8, 256), (8, 256, 8),               # the longest lengths beside the shortest
    (8, 128, 128), (12, 256, 64),           # the largest FP64 planes
    (8, 256, 128), (8, 128, 256),           # FP32 planes whose FP64 ones take the passes
    (8, 24, 192), (8, 192, 24), (8, 96, 192),  # lengths with radix 6 and 12 stages
    (8, 192, 192), (8, 256, 256),  # FP32 planes only; separate passes in both precisions
]


@pytest.mark.parametrize("n", GRIDS)
def test_plane_operators_match_oracle(n):
    from paper_0911_1407_amd.binding import Plan
    inst = synth.make_instance(n, tuple(8.0 * v for v in n), 1.2, 1.1, 1.3, radius=4.0 * n[0], mask_frac=0.2, seed=3,
                               block=2)
    P = oracle_problem(inst)
    rng = np.random.default_rng(6)
    s = inst["s_true"] + 0.05 * rng.standard_normal(n)
    v = rng.standard_normal(n)
    plan = Plan(n, inst["box"], precision="mixed")
    plan.set_instance(inst)
    g, obj = plan.grad(s)
    g_ref, hv_ref = o_model.gradient(P, s), o_model.hessvec(P, s, v)
    assert np.linalg.norm(g.cpu().numpy() - g_ref) <= 1e-11 * np.linalg.norm(g_ref)
    assert_elementwise(g.cpu().numpy(), g_ref, 1e-10, what=f"gradient {n}")
    f_ref = o_model.objective(P, s)
    assert abs(obj - f_ref) <= 1e-11 * abs(f_ref)
    hv = plan.hessvec(v).cpu().numpy()
    assert np.linalg.norm(hv - hv_ref) <= 1e-11 * np.linalg.norm(hv_ref)
    assert_elementwise(hv, hv_ref, 1e-10, what=f"HVP {n}")
    v_hat = np.fft.rfftn(v)
    ref = o_newton.SpectralOps(P).hessvec(o_model.hess_diag(P, s), v_hat)
    vt = torch.from_numpy(v_hat).cuda()
    for dtype, tol in ((torch.complex128, 1e-11), (torch.complex64, 2e-5)):
        out = plan.hessvec_hat(vt.to(dtype)).cpu().numpy()
        assert np.linalg.norm(out - ref) <= tol * np.linalg.norm(ref), dtype
