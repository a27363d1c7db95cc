"""FP64 adjoint solves down to the last digits: the solution's error follows the
tolerance.  The reference refines the same system in torch until its residual
stalls near 4e-16.  From rtol 1e-10 to 1e-12 to 1e-14 the error has to fall by the same
factor 100 each time, within a factor 2 (by how much the last iteration of a
solve passes its tolerance)."""
import math

import numpy as np
import pytest

from paper_0911_1407_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def refined(inst, s, b):
    """lambda with H(s) lambda = b: CG solves to 1e-6 on the residual, repeated."""
    n = inst["n"]
    ncell, vol = n[0] * n[1] * n[2], inst["box"][0] * inst["box"][1] * inst["box"][2]

    def dev(a):
        return torch.as_tensor(a, dtype=torch.float64, device="cuda")

    il = vol / (ncell * inst["amp"] * dev(inst["pk"]))
    il[0, 0, 0] = 0.0
    d = inst["beta"] ** 2 * inst["nbar"] * dev(inst["w"]) * torch.exp(inst["beta"] * dev(s))
    c = torch.full((n[2] // 2 + 1,), 2.0, dtype=torch.float64, device="cuda")
    c[0] = c[-1] = 1.0
    m = 1.0 / (il + torch.quantile(d.flatten(), 0.25).clamp(min=1e-3 * float(d.mean())))

    def hvp(v):
        return il * v + torch.fft.rfftn(d * torch.fft.irfftn(v, s=n))

    def dot(u, v):
        return float(((u.real * v.real + u.imag * v.imag) * c).sum())

    def cg(rhs):
        x, r = torch.zeros_like(rhs), rhs.clone()
        tol2 = 1e-12 * dot(r, r)
        z = m * r
        p, rz = z.clone(), dot(r, z)
        for _ in range(20000):
            q = hvp(p)
            a = rz / dot(p, q)
            x += a * p
            r -= a * q
            if dot(r, r) <= tol2:
                break
            z = m * r
            p, rz = z + (dot(r, z) / rz) * p, dot(r, z)
        return x

    bh = torch.fft.rfftn(dev(b))
    x, bn, last = torch.zeros_like(bh), math.sqrt(dot(bh, bh)), math.inf
    for _ in range(10):
        r = bh - hvp(x)
        rn = math.sqrt(dot(r, r)) / bn
        if rn > 0.5 * last:
            break
        last = rn
        x = x + cg(r)
    assert last < 2e-15
    return torch.fft.irfftn(x, s=n)


@pytest.mark.parametrize("n", [(32, 32, 32), (12, 96, 256)])  # a plane grid, separate passes
def test_error_follows_the_tolerance(n):
    from paper_0911_1407_amd.binding import Plan
    cell = 500.0 / 256
    inst = synth.make_instance(n, tuple(cell * v for v in n), 2.0, 2.0, 1.5, radius=0.4 * cell * max(n), mask_frac=0.2,
                               seed=1, block=4)
    # a field as a reconstruction returns it, and the gradient of a squared
    # error at the observed galaxies
    lam_k = inst["amp"] * inst["pk"] * inst["s_true"].size / np.prod(inst["box"])
    s = np.fft.irfftn(np.fft.rfftn(inst["s_true"]) * lam_k / (lam_k + 0.5), s=n, axes=(0, 1, 2))
    b = 2.0 * inst["counts"] * (s - inst["s_true"])
    lam = refined(inst, s, b)
    plan = Plan(n, inst["box"])
    plan.set_instance(inst)
    err = {}
    for rtol in (1e-10, 1e-12, 1e-14):
        out, info = plan.adjoint(s, b, rtol=rtol, max_cg=30000)
        assert info["status"] == 0, info
        err[rtol] = float((out["lam"] - lam).norm() / lam.norm())
        print(f"{n} rtol {rtol:g}: {info['cg_its']} iterations, error {err[rtol]:.2e}", flush=True)
    assert err[1e-14] <= 0.02 * err[1e-12] <= 0.02 * 0.02 * err[1e-10], err
