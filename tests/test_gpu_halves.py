"""Spectrum columns of padded side 8192, transformed in two half-length parts,
against the float64 split sums: the smallest and the largest side, a side whose rows
end inside a slot, and every multiplier, forward and transposed.  The bars are the
solve's documented ones (1e-6 FP32, 1e-10 FP64)."""
import pytest

import oracle as O
import workloads as W
from test_gpu_pairs import reference

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

COMP = {"x": dict(component="xx"), "y": dict(component="yy"), "xy": dict(component="xy"),
        "coulomb": dict(component="coulomb", partition="erfc"), "gauss": dict(component="coulomb", partition="gauss")}


@pytest.mark.parametrize("n,dtype,component", [
    (2050, torch.float32, "x"), (2050, torch.float64, "y"), (3002, torch.float32, "gauss"),
    (3002, torch.float64, "gauss"), (4094, torch.float32, "coulomb"), (4094, torch.float64, "coulomb"),
    (4096, torch.float32, "xy"), (4096, torch.float64, "x")])
def test_columns_in_halves_against_the_split_sums(n, dtype, component):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_2014_amd as ps
    print(f"case: columns in halves N={n} {dtype} {component}", flush=True)
    half = 16.0
    h = 2 * half / n
    rho = torch.as_tensor(W.mixture_density(n, half, W.draw_mixture(n, 8, 0.375 * half, (0.5, 2.0))), dtype=dtype,
                          device="cuda")
    # rows that differ from their neighbours at the scale of the grid, and both edge rows
    rho[::7] *= 0.25
    rho[0, :] = 0.5
    rho[n - 1, :] = 1.0
    tol, bar = (1e-7, 1e-6) if dtype == torch.float32 else (1e-12, 1e-10)
    kw = dict(component="coulomb", partition="gauss") if component == "gauss" else dict(component=component)
    plan = ps.Plan(n, h, dtype=dtype, tol=tol, **kw)
    got, back = plan.solve(rho), plan.solve_adjoint(rho)
    fine = plan.info["n_fine"]
    plan.close()
    assert fine == 8192
    ref = reference(rho.double(), O.SplitParams(n=n, h=h, n_r=64, n_theta=128, pad_side=fine, **COMP[component]))
    top = ref.abs().max()
    errs = [float((t.double() - ref).abs().max() / top) for t in (got, back)]
    print(f"  rel linf {errs} (bar {bar:.0e})", flush=True)
    assert max(errs) <= bar
