"""The CG's one x pass per iteration (FP64): the solution and the residual it
carries agree after every number of iterations, odd ones included (x takes
the steps of two iterations at once, so an odd count leaves one to add), for
grids with a plane pass and grids without one.  The truncated adjoint solve
returns the iterate and the recurrence's residual norm; the oracle forms the
residual of that iterate.  Tolerance: a handful of iterations accumulate a few
hundred ulp, times the spread of 1/lambda on these coarse cells (below 1e4):
1e-9 of the right-hand side."""
import numpy as np
import pytest

from conftest import oracle_problem
from oracle import model as o_model
from oracle import newton as o_newton
from paper_0911_1407_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [(16, 32, 32), (24, 24, 24), (128, 16, 24)])
def test_iterate_and_residual_agree_at_every_cap(n):
    from paper_0911_1407_amd.binding import Plan
    inst = synth.make_instance(n, tuple(8.0 * v for v in n), 1.2, 1.1, 1.3, radius=4.0 * n[0], mask_frac=0.2, seed=5,
                               block=4)
    P = oracle_problem(inst)
    s = inst["s_true"]
    b = np.random.default_rng(8).standard_normal(n)
    ops, d = o_newton.SpectralOps(P), o_model.hess_diag(P, s)
    b_hat = np.fft.rfftn(b)
    plan = Plan(n, inst["box"])
    plan.set_instance(inst)
    last = np.inf
    for cap in (1, 2, 3, 4, 5, 8, 9):
        out, info = plan.adjoint(s, b, rtol=1e-14, max_cg=cap)
        assert info["cg_its"] == cap
        lam_hat = np.fft.rfftn(out["lam"].cpu().numpy())
        r = b_hat - ops.hessvec(d, lam_hat)
        rel = ops.norm(r) / ops.norm(b_hat)
        assert abs(rel - info["rel_grad"]) <= 1e-9, (cap, rel, info["rel_grad"])
        # the error's H-norm falls with every iteration: lam^H H lam - 2 lam^H b
        f = ops.dot(lam_hat, ops.hessvec(d, lam_hat)) - 2.0 * ops.dot(lam_hat, b_hat)
        assert f < last
        last = f
    # a zero right-hand side: converged at the start, the iterate is zero
    out, info = plan.adjoint(s, np.zeros(n), rtol=1e-10, max_cg=5)
    assert info["cg_its"] == 0 and float(out["lam"].abs().max()) == 0.0
