"""Performance cases: the calls a program that reconstructs density fields makes.

Every case goes through ``Plan`` / ``Batch`` (paper_0911_1407_amd.binding).
Inputs are drawn on the GPU from the seed alone: a lognormal density with the
spectrum P(k) = A k^-1.5 exp(-(2k)^2), a radial selection with whole blocks
masked out, Poisson counts.  ``exact`` recomputes each result with torch in
64 bits (torch.fft, plain Newton and conjugate gradients), without the library.
"""
import math
import os

import torch

from paper_0911_1407_amd import binding
from paper_0911_1407_amd.binding import Batch, Plan

LENGTHS = (8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 512)
BATCH_LENGTHS = (32, 48, 64, 96, 128)
# grids whose schedule the package ships: a program loads it instead of timing
TUNED = {(32, 32, 32), (128, 128, 128), (256, 256, 256), (512, 512, 512)}
TUNE_CACHE = os.path.join(os.path.dirname(os.path.abspath(binding.__file__)), "tune_cache_gfx950.txt")


def listed():
    return [
        # gradient and objective on the small plain grid: one evaluation of an
        # outer sampler or a test, a few launches and a read-back
        _case("grad_plain32", "grad", (32, 32, 32), cell=3.125, sigma=1.0, nbar=1.0),
        # curvature probe (random vector) on a ragged FP64 grid, axes of 2^a and 3 2^a
        _case("hessvec_ragged", "hessvec", (48, 96, 64), cell=3.125, sigma=1.2, nbar=1.0, beta=1.3),
        # the solver's operator on a mid-size cube
        _case("hvp_128", "hvp", (128, 128, 128), cell=2.0, radius=0.4, mask=0.2),
        # the solver's operator on the 256^3 selection workload, FP64 and FP32
        _case("hvp_sel256", "hvp", (256, 256, 256), cell=500.0 / 256, radius=0.4, mask=0.2),
        _case("hvp_sel256_f32", "hvp", (256, 256, 256), cell=500.0 / 256, radius=0.4, mask=0.2, mixed=True),
        # the same operator on the largest grid
        _case("hvp_big512", "hvp", (512, 512, 512), cell=1000.0 / 512, sigma=2.0, nbar=0.2, beta=1.2, radius=0.4),
        # non-local bias: the 13-transform Hessian product on a flat survey slab
        _case("linbias_hessvec", "linbias", (192, 192, 128), cell=3.125, sigma=1.0, nbar=2.0, radius=0.6),
        # a whole MAP reconstruction of the small plain workload
        _case("solve_plain32", "solve", (32, 32, 32), cell=3.125, sigma=1.0, nbar=1.0, rtol=1e-8, hvps=68),
        # the headline reconstruction: 256^3, selection function and mask, FP64,
        # at the default tolerance of the differentiable solve
        _case("solve_sel256", "solve", (256, 256, 256), cell=500.0 / 256, radius=0.4, mask=0.2, rtol=1e-10, hvps=577),
        # the same with FP32 Krylov vectors on a mid-size cube with a power-law bias
        _case("solve_mixed128", "solve", (128, 128, 128), cell=3.125, sigma=1.2, nbar=1.0, beta=1.2, radius=0.5,
              mixed=True, rtol=1e-10, hvps=493),
        # backward pass of the differentiable solve: one adjoint solve
        _case("adjoint_96", "adjoint", (96, 96, 96), cell=3.125, sigma=1.2, nbar=2.0, radius=0.5, rtol=1e-10,
              hvps=193),
        # many small reconstructions of uneven size together, FP32 Krylov vectors
        _case("batch_mixed", "batch", (32, 64, 96), count=16, cell=3.125, sigma=1.2, nbar=1.0, mixed=True, rtol=1e-10,
              hvps=220),
    ]


def _case(name, kind, n, cell, sigma=1.5, nbar=0.5, beta=1.0, radius=0.0, mask=0.0, mixed=False, rtol=0.0, hvps=0,
          count=1):
    c = dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], cell=cell, sigma=sigma, nbar=nbar, beta=beta, radius=radius,
             mask=mask, mixed=mixed, rtol=rtol, hvps=hvps, count=count)
    if name:
        c["name"] = name
    return c


def draw(rng):
    kind = rng.choice(("grad", "hessvec", "hvp", "hvp", "hvp", "hvp", "linbias", "solve", "solve", "adjoint", "batch"))
    # cells spread over the logarithm of the kind's range, axes around the cube root of it
    most = {"grad": 256, "hessvec": 256, "hvp": 512, "linbias": 192, "solve": 128, "adjoint": 96}.get(kind, 96)
    n = [rng.choice([v for v in LENGTHS if 16 <= v <= most])] * 3
    for a in range(3):
        if rng.random() < 0.5:
            near = [v for v in LENGTHS if n[a] / 2 <= v <= min(most, 2 * n[a])]
            n[a] = rng.choice(near)
    c = _case("", kind, n, cell=rng.choice((3.125, 4.0)), sigma=round(rng.uniform(0.8, 1.5), 2),
              nbar=round(math.exp(rng.uniform(math.log(0.3), math.log(3.0))), 3),
              beta=1.0 if kind in ("linbias", "batch") else rng.choice((1.0, 1.2, 1.5)),
              radius=rng.choice((0.0, 0.5)), mixed=kind in ("hvp", "solve", "batch") and rng.random() < 0.5)
    if kind == "hvp":
        c["cell"], c["mask"] = rng.choice((500.0 / 256, 2.0, 3.125)), rng.choice((0.0, 0.2))
    if kind in ("solve", "adjoint", "batch"):
        c["rtol"], c["hvps"] = 1e-10 if c["mixed"] or kind == "adjoint" else 1e-11, {"solve": 400, "adjoint": 200, "batch": 220}[kind]
    if kind == "batch":
        c["nx"], c["ny"], c["nz"] = sorted(rng.choice((32, 48, 64, 96)) for _ in range(3))
        c["count"], c["radius"] = rng.randint(4, 16), 0.0
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _fold(n):
    m = torch.arange(n, device="cuda")
    return torch.where(m >= n // 2, m - n, m).double()


def _power(n, cell):
    """P(k) k-shape on the half spectrum (0 at k = 0); |k| from the integer
    m^2 on cubic boxes, so that the spectrum is exactly isotropic."""
    mx, my, mz = _fold(n[0])[:, None, None], _fold(n[1])[None, :, None], torch.arange(
        n[2] // 2 + 1, device="cuda", dtype=torch.float64)[None, None, :]
    if n[0] == n[1] == n[2]:
        k = torch.sqrt(mx * mx + my * my + mz * mz) * (2 * math.pi / (n[0] * cell))
    else:
        k = torch.sqrt((mx / n[0]) ** 2 + (my / n[1]) ** 2 + (mz / n[2]) ** 2) * (2 * math.pi / cell)
    k[0, 0, 0] = 1.0
    pk = k ** -1.5 * torch.exp(-((2.0 * k) ** 2))
    pk[0, 0, 0] = 0.0
    return pk, k


def _herm(n):
    c = torch.full((n[2] // 2 + 1,), 2.0, dtype=torch.float64, device="cuda")
    c[0] = c[-1] = 1.0
    return c


def _grid_inputs(n, c, gen, sigma=None, nbar=None):
    """One reconstruction problem: prior, selection, counts, the true field."""
    sigma, nbar = sigma or c["sigma"], nbar or c["nbar"]
    pk, _ = _power(n, c["cell"])
    ncell = n[0] * n[1] * n[2]
    vol = ncell * c["cell"] ** 3
    amp = sigma * sigma / (float((pk * _herm(n)).sum()) / vol)
    lam = amp * pk * ncell / vol
    g = torch.randn(n, generator=gen, device="cuda", dtype=torch.float64)
    mu = -0.5 * sigma * sigma
    s_true = torch.fft.irfftn(torch.fft.rfftn(g) * lam.sqrt(), s=n) + mu
    w = torch.ones(n, dtype=torch.float64, device="cuda")
    if c["radius"]:
        ax = [((torch.arange(v, device="cuda", dtype=torch.float64) + 0.5) / v - 0.5) for v in n]
        r2 = ax[0][:, None, None] ** 2 + ax[1][None, :, None] ** 2 + ax[2][None, None, :] ** 2
        w = torch.exp(-r2 / c["radius"] ** 2)
    if c["mask"]:
        nb = [max(1, v // 8) for v in n]
        keep = (torch.rand(nb, generator=gen, device="cuda") >= c["mask"]).double()
        for a in range(3):
            keep = keep.repeat_interleave(n[a] // nb[a], a)
        full = torch.ones(n, dtype=torch.float64, device="cuda")
        full[:keep.shape[0], :keep.shape[1], :keep.shape[2]] = keep
        w = w * full
    counts = torch.poisson(nbar * w * torch.exp(c["beta"] * s_true), generator=gen)
    return dict(n=n, box=tuple(v * c["cell"] for v in n), w=w, counts=counts, pk=pk, amp=amp, mu=mu, nbar=nbar,
                beta=c["beta"], s_true=s_true)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _n(c):
    return (c["nx"], c["ny"], c["nz"])


def _inv_lam(p):
    ncell = p["n"][0] * p["n"][1] * p["n"][2]
    vol = p["box"][0] * p["box"][1] * p["box"][2]
    il = vol / (ncell * p["amp"] * p["pk"])
    il[0, 0, 0] = 0.0
    return il


def _smooth(p):
    """A field as a reconstruction returns it: the true one, Wiener-damped."""
    il = _inv_lam(p)
    sh = torch.fft.rfftn(p["s_true"]) / (1.0 + 0.5 * il)
    return torch.fft.irfftn(sh, s=p["n"]).contiguous()


def _inputs(c, seed):
    """The plain inputs of a case (prepare and exact draw the same ones)."""
    gen = _gen(seed)
    if c["kind"] == "batch":
        sides = (c["nx"], c["ny"], c["nz"])
        out = []
        for i in range(c["count"]):
            u = torch.rand(2, generator=gen, device="cuda").tolist()
            out.append(_grid_inputs((sides[i % 3],) * 3, c, gen, sigma=c["sigma"] * (0.8 + 0.4 * u[0]),
                                    nbar=c["nbar"] * math.exp(u[1] - 0.5)))
        return out
    p = _grid_inputs(_n(c), c, gen)
    if c["kind"] in ("grad", "hvp", "hessvec", "linbias", "adjoint"):
        p["s"] = _smooth(p)
    if c["kind"] in ("hessvec", "linbias"):
        p["v"] = torch.randn(p["n"], generator=gen, device="cuda", dtype=torch.float64)
    if c["kind"] == "hvp":
        # a Krylov direction M^-1 r: M = 1/lambda + const, r white
        r = torch.fft.rfftn(torch.randn(p["n"], generator=gen, device="cuda", dtype=torch.float64))
        p["v_hat"] = (r / (_inv_lam(p) + 0.1)).to(torch.complex64 if c["mixed"] else torch.complex128).contiguous()
    if c["kind"] == "linbias":
        _, k = _power(p["n"], c["cell"])
        k[0, 0, 0] = 0.0
        p["bk"] = 0.9 * torch.exp(-0.5 * (1.5 * k) ** 2)  # below 1: expected counts stay positive
    if c["kind"] == "adjoint":
        p["dL"] = 2.0 * p["counts"] * (p["s"] - p["s_true"])  # squared error at the observed galaxies
    return p


# ---------------------------------------------------------------------------
# the measured calls
# ---------------------------------------------------------------------------

def prepare(case, seed):
    p = _inputs(case, seed)
    if case["kind"] == "batch":
        inst = [dict(q, **{k: q[k].cpu().numpy() for k in ("w", "counts", "pk")}) for q in p]
        b = Batch(inst, precision="mixed" if case["mixed"] else "fp64")
        return dict(kind="batch", batch=b, case=case)
    plan = Plan(p["n"], p["box"], precision="mixed" if case["mixed"] else "fp64")
    plan.set_instance(p)
    if p["n"] in TUNED:
        plan.autotune(TUNE_CACHE)
    st = dict(kind=case["kind"], plan=plan, case=case, **{k: p[k] for k in ("s", "v", "v_hat", "bk", "dL") if k in p})
    if case["kind"] in ("hvp", "hessvec"):
        plan.hessvec(torch.zeros_like(p["s"]), s=p["s"])  # linearise at s: later products reuse the diagonal
    if case["kind"] == "linbias":
        st["grad"], _ = plan.linear_bias_grad("lognormal", p["bk"], p["s"])
    return st


def run(st):
    plan, c, kind = st.get("plan"), st["case"], st["kind"]
    if kind == "grad":
        g, obj = plan.grad(st["s"])
        return {"grad": g, "obj": obj}
    if kind == "hessvec":
        return plan.hessvec(st["v"])
    if kind == "hvp":
        return plan.hessvec_hat(st["v_hat"])
    if kind == "linbias":
        return plan.linear_bias_hessvec("lognormal", st["bk"], st["v"])
    if kind == "solve":
        s, _ = plan.solve(rtol=c["rtol"], precision=1 if c["mixed"] else 0)
        return s
    if kind == "adjoint":
        out, _ = plan.adjoint(st["s"], st["dL"], rtol=c["rtol"], max_cg=20000)
        return out
    s, _ = st["batch"].solve(rtol=c["rtol"], precision=1 if c["mixed"] else 0)
    return s


def work(case):
    """Bytes and operations no implementation avoids: an operator reads its
    vector, the diagonal (for a gradient the data) and writes its result; a
    solve does that once per Hessian product.  Half spectra count as real
    fields; a 3D real transform takes 2.5 N log2 N operations."""
    if case["kind"] == "batch":
        sides = (case["nx"], case["ny"], case["nz"])
        cells = [sides[i % 3] ** 3 for i in range(case["count"])]
    else:
        cells = [case["nx"] * case["ny"] * case["nz"]]
    e = 4 if case["mixed"] else 8
    fields = {"grad": 4, "hessvec": 3, "hvp": 3, "linbias": 5}.get(case["kind"], 3) * e
    ffts = {"linbias": 6}.get(case["kind"], 2)
    reps = max(1, case["hvps"])
    return {"bytes": float(sum(cells) * fields * reps),
            "flops": float(sum(v * (ffts * 2.5 * math.log2(v) + 8) for v in cells) * reps)}


# ---------------------------------------------------------------------------
# the same results in plain 64-bit torch
# ---------------------------------------------------------------------------

class _Spectral:
    def __init__(self, p):
        self.n, self.N = p["n"], p["n"][0] * p["n"][1] * p["n"][2]
        self.il, self.c = _inv_lam(p), _herm(p["n"])

    def fwd(self, x):
        return torch.fft.rfftn(x)

    def inv(self, x):
        return torch.fft.irfftn(x, s=self.n)

    def dot(self, a, b):
        return float(((a.real * b.real + a.imag * b.imag) * self.c).sum()) / self.N

    def hvp(self, d, v):
        return self.il * v + self.fwd(d * self.inv(v))

    def cg(self, d, rhs, tol, most):
        low = torch.quantile(d.flatten()[::max(1, self.N // 1000000)], 0.25)
        m = 1.0 / (self.il + low.clamp(min=1e-3 * float(d.mean())))
        x, r = torch.zeros_like(rhs), rhs.clone()
        z = m * r
        p, rz = z.clone(), self.dot(r, z)
        for _ in range(most):
            q = self.hvp(d, p)
            a = rz / self.dot(p, q)
            x += a * p
            r -= a * q
            if math.sqrt(self.dot(r, r)) <= tol:
                break
            z = m * r
            new = self.dot(r, z)
            p, rz = z + (new / rz) * p, new
        return x


def _map(p, rtol):
    """MAP by Newton's method on the half spectrum (Armijo backtracking)."""
    o, beta, nbar, w, cnt = _Spectral(p), p["beta"], p["nbar"], p["w"], p["counts"]
    x = torch.zeros_like(o.il, dtype=torch.complex128)  # spectrum of s - mu

    def lin(x):
        s = o.inv(x) + p["mu"]
        e = nbar * w * torch.exp(beta * s)
        return s, e, o.il * x + o.fwd(beta * (e - cnt))

    s, e, g = lin(x)
    g0 = gn = math.sqrt(o.dot(g, g))
    for _ in range(60):
        if gn <= rtol * g0:
            break
        eta = min(0.3, max(gn / g0, 0.3 * rtol * g0 / gn))
        h = o.cg(beta * beta * e, -g, eta * gn, 800)
        hr, b, c2, slope, a = o.inv(h), o.dot(h, o.il * x), o.dot(h, o.il * h), o.dot(g, h), 1.0
        for _ in range(30):
            df = a * b + 0.5 * a * a * c2 + float((e * torch.expm1(a * beta * hr) - a * beta * cnt * hr).sum())
            if df <= 1e-4 * a * slope:
                break
            a *= 0.5
        x = x + a * h
        s, e, g = lin(x)
        gn = math.sqrt(o.dot(g, g))
    return s


def exact(case, seed):
    p = _inputs(case, seed)
    kind = case["kind"]
    if kind == "batch":
        return [_map(q, 1e-12) for q in p]
    if kind == "solve":
        return _map(p, 1e-12)
    o = _Spectral(p)
    beta, s = p["beta"], p["s"]
    e = p["nbar"] * p["w"] * torch.exp(beta * s)
    d = beta * beta * e
    if kind == "grad":
        xs = o.fwd(s - p["mu"])
        obj = 0.5 * o.dot(xs, o.il * xs) + float((e - beta * p["counts"] * s).sum())
        return {"grad": o.inv(o.il * xs) + beta * (e - p["counts"]), "obj": obj}
    if kind == "hessvec":
        return o.inv(o.il * o.fwd(p["v"])) + d * p["v"]
    if kind == "hvp":
        return o.hvp(d, p["v_hat"].to(torch.complex128))
    if kind == "linbias":
        conv = lambda f: o.inv(p["bk"] * o.fwd(f))  # noqa: E731
        y, es, v = 1.0 + conv(torch.expm1(s)), torch.exp(s), p["v"]
        u = p["nbar"] * p["w"] - p["counts"] / y
        return o.inv(o.il * o.fwd(v)) + es * conv(u) * v + es * conv(p["counts"] / (y * y) * conv(es * v))
    # adjoint
    b = o.fwd(p["dL"])
    lam = o.inv(o.cg(d, b, 1e-13 * math.sqrt(o.dot(b, b)), 6000))
    ebs = torch.exp(beta * s)
    prior = o.il * o.fwd(s - p["mu"])
    return {"A": o.dot(o.fwd(lam), prior) / p["amp"],
            "beta": -float((lam * (e * (1.0 + beta * s) - p["counts"])).sum()),
            "nbar": -float((lam * beta * p["w"] * ebs).sum()),
            "N": beta * lam, "w": -lam * beta * p["nbar"] * ebs, "lam": lam}
