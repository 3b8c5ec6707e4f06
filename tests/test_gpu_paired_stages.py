"""The type-2 and type-1 stages, and solves with the Gaussian kernel, where the rows
run in pairs: padded sides from 2048 (FP32) and 4096 (FP64) whose deconvolution
series is short (small for wide boxes and loose tolerances, its coefficients up to
120 times the factors' for the Gaussian kernel).  The stages run on every node, the
solves on one half plane.  Bars: 10 tol in relative l2 for a stage, on smooth and on
independent random values; 1e-6 (FP32) and 1e-10 (FP64) for a solve.  The
references are the direct sums in float64, with torch on the GPU."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from test_gpu_pairs import reference

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

HALF = 16.0


def density(kind, n, dtype):
    if kind == "noise":
        gen = torch.Generator(device="cuda").manual_seed(n)
        return torch.randn((n, n), dtype=dtype, device="cuda", generator=gen)
    spec = W.draw_mixture(n, 8, 0.375 * HALF, (0.5, 2.0))
    return torch.as_tensor(W.mixture_density(n, HALF, spec), dtype=dtype, device="cuda")


def phases(plan, n):
    """e^{-2 pi i k x} of every node and grid point, along x and along y."""
    dev = {"device": "cuda", "dtype": torch.float64}
    x = torch.as_tensor(O.grid_points(O.SplitParams(n, 2 * HALF / n, 1, 2)), **dev)
    kx, ky = (torch.as_tensor(a, **dev) for a in plan.nodes()[:2])
    return [torch.polar(torch.ones_like(a), -2 * np.pi * a) for a in (torch.outer(kx, x), torch.outer(ky, x))]


CASES = [(514, torch.float32, 1e-7), (1024, torch.float32, 1e-4), (1026, torch.float32, 1e-7),
         (2050, torch.float32, 1e-7), (1026, torch.float64, 1e-12), (1500, torch.float64, 1e-9),
         (2050, torch.float64, 1e-12)]


@pytest.mark.parametrize("kernel", ["es", "gaussian"])
@pytest.mark.parametrize("kind", ["smooth", "noise"])
@pytest.mark.parametrize("n,dtype,tol", CASES)
def test_stages_on_paired_rows(n, dtype, tol, kind, kernel):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_2014_amd as ps
    print(f"case: stages on paired rows N={n} {dtype} tol={tol} {kind} {kernel}", flush=True)
    h = 2 * HALF / n
    plan = ps.Plan(n, h, dtype=dtype, tol=tol, n_r=16, n_theta=64, kernel=kernel)
    ex, ey = phases(plan, n)
    rho = density(kind, n, dtype)
    hat = ((ey @ rho.to(torch.complex128)) * ex).sum(1) * h * h
    got2 = plan.type2(rho).to(torch.complex128)
    if kind == "noise":
        gen = torch.Generator(device="cuda").manual_seed(n + 1)
        coef = torch.view_as_complex(torch.randn((hat.numel(), 2), dtype=torch.float64, device="cuda", generator=gen))
    else:
        coef = torch.as_tensor(plan.nodes()[2], device="cuda") * hat
    coef = coef.to(torch.complex64 if dtype == torch.float32 else torch.complex128)
    field = (ey.conj().resolve_conj().T.contiguous() @ (ex.conj().resolve_conj() * coef.to(torch.complex128)[:, None])).real
    got1 = plan.type1(coef).double()
    plan.close()
    errs = [float((a - b).norm() / b.norm()) for a, b in ((got2, hat), (got1, field))]
    print(f"  rel l2 type 2 {errs[0]:.2e}, type 1 {errs[1]:.2e} (bar {10 * tol:.0e})", flush=True)
    assert max(errs) <= 10 * tol


@pytest.mark.parametrize("n,dtype,tol,component", [
    (514, torch.float32, 1e-7, "x"), (1026, torch.float32, 1e-7, "xy"), (2050, torch.float32, 1e-7, "coulomb"),
    (1026, torch.float64, 1e-12, "x"), (2050, torch.float64, 1e-12, "y")])
def test_gaussian_kernel_on_paired_rows(n, dtype, tol, component):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_2014_amd as ps
    print(f"case: Gaussian kernel on paired rows N={n} {dtype} {component}", flush=True)
    h = 2 * HALF / n
    rho = density("smooth", n, dtype)
    plan = ps.Plan(n, h, dtype=dtype, tol=tol, component=component, kernel="gaussian")
    got, back = plan.solve(rho), plan.solve_adjoint(rho)
    fine = plan.info["n_fine"]
    plan.close()
    comp = {"x": "xx", "y": "yy", "xy": "xy", "coulomb": "coulomb"}[component]
    part = {"partition": "erfc"} if component == "coulomb" else {}
    ref = reference(rho.double(), O.SplitParams(n=n, h=h, n_r=64, n_theta=128, pad_side=fine, component=comp, **part))
    errs = [float((t.double() - ref).abs().max() / ref.abs().max()) for t in (got, back)]
    bar = 1e-6 if dtype == torch.float32 else 1e-10
    print(f"  rel linf {errs} (bar {bar:.0e})", flush=True)
    assert max(errs) <= bar
