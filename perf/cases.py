"""The work that users of this package have it do, as timed cases.

Each case is one call chain through the public entry points: single solves and
transposed solves from 64^2 to 3000^2 in both precisions (power-of-two and
ragged sides, every multiplier), the differentiable solve, uneven batches, the
periodic solver, and the DS time stepper forward and with its checkpointed
gradient.  Densities are |u|^2 of seeded sums of eight anisotropic complex
Gaussians, the package's own workload shape.

A case has a "kind" and its sizes:

  solve      Plan.solve (or .solve_adjoint), called eagerly
  replay     forward + transposed solve captured once in a HIP graph (as a serving
             loop keeps it), one replay per pass
  grad       phi_solve through autograd: the potential and the gradient of
             ||Phi - target||^2 in the density
  batch      BatchPlan.solve (or .solve_adjoint) over members of uneven sides
  periodic   Plan.periodic, the standard periodic FFT solver
  steps      DSStepper.forward, a few split steps of a complex field
  stepgrad   DSStepper.loss_and_grad with checkpoints
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_1409_2014_amd as ps

LOG_INV_EPS = math.log(1e16)     # fixes the default partition width and disk radius


def listed():
    return [
        # the smallest example of the paper (Sec. 3.1): latency and launches count
        {"name": "solve_64_f64", "kind": "solve", "n": 64, "half": 8.0, "dtype": "f64", "n_r": 32, "n_theta": 64,
         "component": "x", "adjoint": False},
        # a ragged side between two padded ones, transposed: the general grid bounds
        {"name": "adjoint_300_f64", "kind": "solve", "n": 300, "half": 8.0, "dtype": "f64", "n_r": 64, "n_theta": 128,
         "component": "x", "adjoint": True},
        # the Coulomb multiplier at an ordinary size
        {"name": "coulomb_512_f32", "kind": "solve", "n": 512, "half": 8.0, "dtype": "f32", "n_r": 64, "n_theta": 128,
         "component": "coulomb", "adjoint": False},
        # a captured pair at a small side, as an optimisation loop replays it
        {"name": "replay_256_f32", "kind": "replay", "n": 256, "half": 8.0, "dtype": "f32", "n_r": 64, "n_theta": 128,
         "component": "x"},
        # the headline size in both precisions, replayed
        {"name": "replay_2048_f32", "kind": "replay", "n": 2048, "half": 16.0, "dtype": "f32", "n_r": 64,
         "n_theta": 128, "component": "x"},
        {"name": "replay_2048_f64", "kind": "replay", "n": 2048, "half": 16.0, "dtype": "f64", "n_r": 64,
         "n_theta": 128, "component": "x"},
        # the largest: a ragged side on the 8192 padded box, the mixed multiplier
        {"name": "solve_3000_xy_f32", "kind": "solve", "n": 3000, "half": 24.0, "dtype": "f32", "n_r": 64,
         "n_theta": 128, "component": "xy", "adjoint": False},
        # the differentiation workload
        {"name": "grad_1024_f64", "kind": "grad", "n": 1024, "half": 16.0, "dtype": "f64", "n_r": 64, "n_theta": 128,
         "component": "x"},
        # an uneven batch of the benchmark's sides, and a ragged one, transposed
        {"name": "batch_64_f32", "kind": "batch", "count": 64, "lo": 128, "hi": 1024, "pow2": True, "dtype": "f32",
         "adjoint": False},
        {"name": "batch_12_ragged_f64", "kind": "batch", "count": 12, "lo": 130, "hi": 700, "pow2": False,
         "dtype": "f64", "adjoint": True},
        # time stepping at the benchmark's size, and a checkpointed gradient
        {"name": "steps_2048_f32", "kind": "steps", "n": 2048, "half": 32.0, "dtype": "f32", "steps": 20,
         "scheme": "strang", "potential": "split"},
        {"name": "stepgrad_512_f64", "kind": "stepgrad", "n": 512, "half": 16.0, "dtype": "f64", "steps": 4,
         "every": 2, "scheme": "strang", "potential": "split"},
    ]


def _even(rng: random.Random, lo: int, hi: int) -> int:
    """An even side, spread over the logarithm of the range."""
    return 2 * int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / 2))


def draw(rng: random.Random):
    kind = rng.choice(["solve", "solve", "solve", "replay", "grad", "batch", "periodic", "steps", "stepgrad"])
    dtype = rng.choice(["f32", "f64"])
    n_r, n_theta = rng.choice([(32, 64), (64, 128), (60, 60)])
    if kind in ("solve", "replay", "grad"):
        n = _even(rng, 64, 3000 if dtype == "f32" else 2048)
        if rng.random() < 0.4:       # much of all use is on power-of-two sides
            n = min(2048, 1 << int(round(math.log2(n))))
        c = {"kind": kind, "n": n, "half": rng.choice([8.0, 12.0, 16.0, 24.0]), "dtype": dtype, "n_r": n_r,
             "n_theta": n_theta, "component": rng.choice(["x", "x", "x", "y", "xy", "coulomb"])}
        if kind == "solve":
            c["adjoint"] = rng.random() < 0.4
        return c
    if kind == "batch":
        lo = rng.choice([66, 100, 128, 200])
        return {"kind": "batch", "count": rng.randrange(3, 25), "lo": lo, "hi": rng.choice([300, 512, 700, 1024]),
                "pow2": rng.random() < 0.5, "dtype": dtype, "adjoint": rng.random() < 0.5}
    if kind == "periodic":
        return {"kind": "periodic", "n": 1 << rng.randrange(6, 12), "half": rng.choice([16.0, 32.0]), "dtype": dtype,
                "component": rng.choice(["x", "y", "xy"])}
    n = 1 << rng.randrange(6, 11 if kind == "steps" else 10)
    c = {"kind": kind, "n": n, "half": rng.choice([12.0, 16.0]), "dtype": dtype, "steps": rng.randrange(1, 6),
         "scheme": rng.choice(["strang", "yoshida4"]), "potential": rng.choice(["split", "split", "periodic"])}
    if kind == "stepgrad":
        c["every"] = rng.randrange(1, 4)
    return c


# ---- inputs ------------------------------------------------------------------
def _real(case):
    return torch.float32 if case["dtype"] == "f32" else torch.float64


def _wave(n: int, half: float, seed: int) -> torch.Tensor:
    """A sum of eight anisotropic complex Gaussians on [-half, half)^2, complex128 on the GPU."""
    rng = np.random.default_rng(seed)
    cx, cy = rng.uniform(-0.375 * half, 0.375 * half, (2, 8))
    wx, wy = rng.uniform(0.5, 2.0, (2, 8)) * (half / 16.0)
    ph = rng.uniform(0.0, 2.0 * math.pi, 8)
    x = -half + (2.0 * half / n) * np.arange(n)
    gx = np.exp(-((x[None] - cx[:, None]) / wx[:, None]) ** 2)
    gy = np.exp(-((x[None] - cy[:, None]) / wy[:, None]) ** 2) * np.exp(1j * ph)[:, None]
    gx = torch.as_tensor(gx, device="cuda").to(torch.complex128)
    gy = torch.as_tensor(gy, device="cuda")
    return (gy.T.contiguous() @ gx).contiguous()


def _density(n: int, half: float, seed: int, dtype) -> torch.Tensor:
    u = _wave(n, half, seed)
    return (u.real ** 2 + u.imag ** 2).to(dtype).contiguous()


def _tol(case):
    return 1e-7 if case["dtype"] == "f32" else 1e-12


def _members(case):
    """(side, box half-width) of a batch's members: h = 1/32, sides fixed by the case."""
    rng = random.Random(case["count"] * 1009 + case["lo"] * 31 + case["hi"])
    out = []
    for _ in range(case["count"]):
        n = _even(rng, case["lo"], case["hi"])
        if case["pow2"]:
            n = min(1024, max(128, 1 << int(round(math.log2(n)))))
        out.append((n, n / 64.0))
    return out


def _field(case, seed):
    """A field of unit size and moderate frequencies for the stepper."""
    u = _wave(case["n"], case["half"], seed)
    return (u / u.abs().max()).to(torch.complex64 if case["dtype"] == "f32" else torch.complex128).contiguous()


def _plan(case):
    return ps.Plan(case["n"], 2.0 * case["half"] / case["n"], dtype=_real(case), n_r=case["n_r"],
                   n_theta=case["n_theta"], tol=_tol(case), component=case["component"])


def prepare(case, seed):
    kind, dtype = case["kind"], _real(case)
    st = {"case": case}
    if kind == "batch":
        members = _members(case)
        st["plan"] = ps.BatchPlan([dict(n=n, h=2.0 * half / n, n_r=64, n_theta=128, tol=_tol(case))
                                   for n, half in members], dtype=dtype)
        st["rho"] = st["plan"].pack([_density(n, half, seed * 1000 + i, dtype) for i, (n, half) in enumerate(members)])
        st["out"] = torch.empty_like(st["rho"])
    elif kind in ("steps", "stepgrad"):
        st["plan"] = ps.DSStepper(case["n"], 2.0 * case["half"] / case["n"], tau=1e-3, dtype=dtype,
                                  scheme=case["scheme"], potential=case["potential"], tol=_tol(case))
        st["u0"] = _field(case, seed)
        st["u"] = torch.empty_like(st["u0"])
    elif kind == "periodic":
        st["plan"] = ps.Plan(case["n"], 2.0 * case["half"] / case["n"], dtype=dtype, component=case["component"])
        st["rho"] = _density(case["n"], case["half"], seed, dtype)
        st["out"] = torch.empty_like(st["rho"])
    else:
        st["plan"] = _plan(case)
        st["rho"] = _density(case["n"], case["half"], seed, dtype)
        st["out"] = torch.empty_like(st["rho"])
        if kind == "grad":
            st["target"] = _density(case["n"], case["half"], seed + 1, dtype)
            st["rho"].requires_grad_(True)
        if kind == "replay":
            st["back"] = torch.empty_like(st["rho"])
            plan, side = st["plan"], torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                plan.solve(st["rho"], st["out"])
                plan.solve_adjoint(st["out"], st["back"])
            torch.cuda.current_stream().wait_stream(side)
            st["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(st["graph"]):
                plan.solve(st["rho"], st["out"])
                plan.solve_adjoint(st["out"], st["back"])
    return st


def run(st):
    case, plan = st["case"], st["plan"]
    kind = case["kind"]
    if kind in ("solve", "batch"):
        return (plan.solve_adjoint if case["adjoint"] else plan.solve)(st["rho"], st["out"])
    if kind == "replay":
        st["graph"].replay()
        return st["out"], st["back"]
    if kind == "grad":
        phi = ps.phi_solve(st["rho"], plan)
        grad, = torch.autograd.grad(((phi - st["target"]) ** 2).sum(), st["rho"])
        return phi.detach(), grad
    if kind == "periodic":
        return plan.periodic(st["rho"], st["out"])
    if kind == "steps":
        st["u"].copy_(st["u0"])
        return plan.forward(st["u"], case["steps"])
    loss, grad, _ = plan.loss_and_grad(st["u0"], case["steps"], case["every"])
    return loss, grad


# ---- the work a pass cannot do without ---------------------------------------
def _padded(n: int) -> int:
    f = 16
    while f < 2 * n:
        f *= 2
    return f


def _solve_work(n, es, nodes, width):
    """Density read, potential written; a zero-padded real 2-D transform and its
    inverse (only the rows and columns that hold data), and the node sums."""
    f = _padded(n)
    lg = math.log2(f)
    flops = 2 * (n * 2.5 * f * lg + (f / 2 + 1) * 5.0 * f * lg) + 2 * nodes * width * width * 4.0
    return {"bytes": 2.0 * n * n * es, "flops": flops}


def _periodic_work(n, es):
    lg = math.log2(n)
    return {"bytes": 2.0 * n * n * es, "flops": 2 * (n * 2.5 * n * lg + (n / 2 + 1) * 5.0 * n * lg)}


def _steps_work(case, solves, flows):
    n, es = case["n"], 4 if case["dtype"] == "f32" else 8
    one = _periodic_work(n, es) if case["potential"] == "periodic" else _solve_work(n, es, 8192, 8 if es == 4 else 13)
    flow = 2 * 2 * n * 5.0 * n * math.log2(n)
    return {"bytes": 2.0 * 2 * n * n * es, "flops": solves * one["flops"] + flows * flow}


def work(case):
    kind, es = case["kind"], 4 if case["dtype"] == "f32" else 8
    width = 8 if es == 4 else 13
    if kind == "batch":
        parts = [_solve_work(n, es, 8192, width) for n, _ in _members(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    if kind == "periodic":
        return _periodic_work(case["n"], es)
    if kind in ("steps", "stepgrad"):
        sub = 3 if case["scheme"] == "yoshida4" else 1
        solves = sub * case["steps"]
        if kind == "steps":
            return _steps_work(case, solves, solves + 1)
        # forward, recomputed segments but the last, transposed
        last = case["steps"] % case["every"] or case["every"]
        total = solves + sub * (case["steps"] - min(last, case["steps"])) + solves
        return _steps_work(case, total, total + 2)
    w = _solve_work(case["n"], es, case["n_r"] * case["n_theta"], width)
    return {k: v * (1 if kind == "solve" else 2) for k, v in w.items()}


# ---- the same outputs in 64 bits, from the formulas ----------------------------
def _multiplier(component, kx, ky):
    """(-k_a k_b / |k|^2 with 0 at the origin, |k|^2)."""
    k2 = kx * kx + ky * ky
    num = {"x": kx * kx, "y": ky * ky, "xy": kx * ky}[component]
    return -num / torch.where(k2 > 0, k2, torch.ones_like(k2)), k2


class _Exact:
    """Phi for one grid: the zero-padded trapezoidal sum for the high frequencies
    plus the polar quadrature with direct nonuniform sums, in float64."""

    def __init__(self, n, half, n_r, n_theta, component):
        self.n, self.f = n, _padded(n)
        h = 2.0 * half / n
        f = self.f
        sigma = math.sqrt(LOG_INV_EPS) / (2.0 * math.pi * (f / n - 1.0) * half)
        cut = math.sqrt(LOG_INV_EPS) * sigma
        dev = {"device": "cuda", "dtype": torch.float64}
        kx = (torch.arange(f // 2 + 1, **dev) / (f * h))[None, :]
        m = torch.arange(f, **dev)
        ky = (torch.where(m < f // 2, m, m - f) / (f * h))[:, None]
        if component == "coulomb":
            k = torch.sqrt(kx * kx + ky * ky)
            g = torch.erf(k / sigma) / torch.where(k > 0, k, torch.ones_like(k))
            g[0, 0] = 2.0 / (sigma * math.sqrt(math.pi))
        else:
            mult, k2 = _multiplier(component, kx, ky)
            g = mult * -torch.expm1(-k2 / sigma ** 2)
            if component == "xy":      # a bin on a Nyquist line stands for +k and -k
                g[:, f // 2] = 0.0
                g[f // 2, :] = 0.0
        self.g = g
        x, w = np.polynomial.legendre.leggauss(n_r)
        r = 0.5 * cut * (1.0 + x)
        th = 2.0 * math.pi * np.arange(n_theta) / n_theta
        if component == "coulomb":
            radial = 0.5 * cut * w * np.array([math.erfc(v / sigma) for v in r])
            ang = np.ones_like(th)
        else:
            radial = -0.5 * cut * w * r * np.exp(-(r / sigma) ** 2)
            ang = {"x": np.cos(th) ** 2, "y": np.sin(th) ** 2, "xy": np.cos(th) * np.sin(th)}[component]
        q = np.outer(radial, ang * (2.0 * math.pi / n_theta)).ravel()
        pts = -half + h * np.arange(n)
        as_t = lambda a: torch.as_tensor(a, **dev)   # noqa: E731
        self.q = as_t(q * h * h)
        ax = 2.0 * math.pi * torch.outer(as_t(np.outer(r, np.cos(th)).ravel()), as_t(pts))
        ay = 2.0 * math.pi * torch.outer(as_t(np.outer(r, np.sin(th)).ravel()), as_t(pts))
        self.ex = torch.polar(torch.ones_like(ax), -ax)      # [node][x]
        self.ey = torch.polar(torch.ones_like(ay), -ay)

    def __call__(self, rho):
        n, f = self.n, self.f
        i1 = torch.fft.irfft2(torch.fft.rfft2(rho, s=(f, f)) * self.g, s=(f, f))[:n, :n]
        at = ((self.ey @ rho.to(torch.complex128)) * self.ex).sum(1) * self.q
        eyc = torch.conj(self.ey).resolve_conj().T.contiguous()
        exc = torch.conj(self.ex).resolve_conj()
        return i1 + (eyc @ (exc * at[:, None])).real


class _ExactPeriodic:
    def __init__(self, n, half, component):
        k = torch.fft.fftfreq(n, device="cuda", dtype=torch.float64) * n
        self.n = n
        kx = k[None, :]
        ky = k[:, None]
        self.g, _ = _multiplier(component, kx, ky)
        self.g[0, 0] = 0.0
        if component == "xy":
            self.g[:, n // 2] = 0.0
            self.g[n // 2, :] = 0.0

    def __call__(self, rho):
        return torch.fft.ifft2(torch.fft.fft2(rho.to(torch.complex128)) * self.g).real


def _evolve(case, potential, u, steps, tau=1e-3):
    """Strang or fourth-order split steps of i u_t = (-d_xx + d_yy) u with the
    phase tau (2 |u|^2 + 4 Phi) of the nonlinear substep."""
    n, h = case["n"], 2.0 * case["half"] / case["n"]
    k = torch.fft.fftfreq(n, d=h, device="cuda", dtype=torch.float64)
    w = 4.0 * math.pi ** 2 * ((k ** 2)[None, :] - (k ** 2)[:, None])
    if case["scheme"] == "strang":
        parts = [(0.5, 1.0), (0.5, None)]
    else:
        b1 = 1.0 / (2.0 - 2.0 ** (1.0 / 3.0))
        b2 = 1.0 - 2.0 * b1
        parts = [(b1 / 2, b1), ((b1 + b2) / 2, b2), ((b1 + b2) / 2, b1), (b1 / 2, None)]
    for _ in range(steps):
        for a, b in parts:
            u = torch.fft.ifft2(torch.fft.fft2(u) * torch.polar(torch.ones_like(w), -w * (a * tau)))
            if b is not None:
                rho = u.real ** 2 + u.imag ** 2
                ph = b * tau * (2.0 * rho + 4.0 * potential(rho))
                u = u * torch.polar(torch.ones_like(ph), ph)
    return u


def exact(case, seed):
    kind, dtype = case["kind"], _real(case)
    if kind == "batch":
        out = []
        for i, (n, half) in enumerate(_members(case)):
            rho = _density(n, half, seed * 1000 + i, dtype).double()
            out.append(_Exact(n, half, 64, 128, "x")(rho).reshape(-1))
        return torch.cat(out)
    if kind == "periodic":
        return _ExactPeriodic(case["n"], case["half"], case["component"])(
            _density(case["n"], case["half"], seed, dtype).double())
    if kind in ("steps", "stepgrad"):
        pot = (_ExactPeriodic(case["n"], case["half"], "x") if case["potential"] == "periodic"
               else _Exact(case["n"], case["half"], 64, 128, "x"))
        u = _field(case, seed).to(torch.complex128)
        if kind == "steps":
            return _evolve(case, pot, u, case["steps"])
        u.requires_grad_(True)
        h = 2.0 * case["half"] / case["n"]
        v = _evolve(case, pot, u, case["steps"])
        loss = h * h * ((v.real ** 2 + v.imag ** 2) ** 2).sum()
        grad, = torch.autograd.grad(loss, u)
        return loss.detach(), grad
    rho = _density(case["n"], case["half"], seed, dtype).double()
    phi = _Exact(case["n"], case["half"], case["n_r"], case["n_theta"], case["component"])
    first = phi(rho)
    if kind == "solve":
        return first        # the operator is symmetric: the transposed solve is the same sum
    if kind == "replay":
        return first, phi(first)
    target = _density(case["n"], case["half"], seed + 1, dtype).double()
    return first, phi(2.0 * (first - target))
