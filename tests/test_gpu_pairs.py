"""Solves whose rows run in pairs (padded side 2048 and up in FP32, 4096 and up in
FP64) against the float64 split sums, forward and transposed: sides at both ends
of a padded side, numbers of pairs that the pairs per block do not divide,
multipliers, and tolerances whose deconvolution series has few terms, many, or
none that is accurate (the one-row kernels then serve the plan).  The reference
is evaluated with torch on the GPU in float64, from the oracle's nodes, weights
and multiplier."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def reference(rho, p):
    """Phi in float64: the oracle's sums as torch matrix products."""
    dev = {"device": "cuda", "dtype": torch.float64}
    n, m = p.n, p.padded_side
    g = torch.as_tensor(O.split_solver.padded_multiplier(p), **dev)
    i1 = torch.fft.ifft2(torch.fft.fft2(rho, s=(m, m)) * g)[:n, :n].real
    kx, ky, q = (torch.as_tensor(np.ravel(a), **dev) for a in O.polar_rule(p))
    x = torch.as_tensor(O.grid_points(p), **dev)
    ex, ey = (torch.polar(torch.ones_like(a), -2 * np.pi * a) for a in (torch.outer(kx, x), torch.outer(ky, x)))
    c = ((ey @ rho.to(torch.complex128)) * ex).sum(1) * q * p.h ** 2
    return i1 + (ey.conj().resolve_conj().T.contiguous() @ (ex.conj().resolve_conj() * c[:, None])).real


# (n, half, dtype, tol, component, bar): the bar is the solve's documented one
# (1e-6 FP32, 1e-10 FP64) or 20 tol where the tolerance is looser
CASES = [
    (514, 8.0, torch.float32, 1e-7, "x", 1e-6),
    (1022, 16.0, torch.float32, 1e-7, "xy", 1e-6),
    (1024, 16.0, torch.float32, 1e-2, "x", 0.2),
    (1026, 16.0, torch.float32, 1e-7, "y", 1e-6),
    (1026, 16.0, torch.float64, 1e-12, "x", 1e-10),
    (2048, 16.0, torch.float64, 1e-6, "x", 2e-5),
    (2048, 16.0, torch.float64, 1e-15, "x", 1e-10),
    (2046, 16.0, torch.float64, 1e-12, "coulomb", 1e-10),
    (2050, 16.0, torch.float32, 1e-7, "x", 1e-6),
]


@pytest.mark.parametrize("n,half,dtype,tol,component,bar", CASES)
def test_paired_rows_against_the_split_sums(n, half, dtype, tol, component, bar):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_2014_amd as ps
    print(f"case: paired rows N={n} {dtype} tol={tol} {component}", flush=True)
    h = 2 * half / n
    rho = torch.as_tensor(W.mixture_density(n, half, W.draw_mixture(n, 8, 0.375 * half, (0.5, 2.0))), dtype=dtype,
                          device="cuda")
    # rows that differ from their neighbours at the scale of the grid, and an edge row
    rho[::7] *= 0.25
    rho[n - 1, :] = 1.0
    plan = ps.Plan(n, h, dtype=dtype, tol=tol, component=component)
    got, back = plan.solve(rho), plan.solve_adjoint(rho)
    parts = plan.highfreq(rho).double() + plan.lowfreq(rho).double()
    fine = plan.info["n_fine"]
    plan.close()
    comp = {"x": "xx", "y": "yy", "xy": "xy", "coulomb": "coulomb"}[component]
    part = {"partition": "erfc"} if component == "coulomb" else {}
    ref = reference(rho.double(), O.SplitParams(n=n, h=h, n_r=64, n_theta=128, pad_side=fine, component=comp, **part))
    top = ref.abs().max()
    errs = [float((t.double() - ref).abs().max() / top) for t in (got, back, parts)]
    print(f"  rel linf {errs} (bar {bar:.0e})", flush=True)
    assert max(errs) <= bar
