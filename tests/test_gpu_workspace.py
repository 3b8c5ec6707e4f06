"""Device memory of plans: which plans phi_solve_noalloc's static scratch takes,
and what a batch plan holds."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# workspaces just below the 80 MiB of the scratch, with kernels narrower than 13 cells
@pytest.mark.parametrize("n,dtype,kw", [
    (2394, torch.float32, dict(n_r=128, n_theta=256, tol=1e-7)),
    (2412, torch.float32, dict(n_r=64, n_theta=128, tol=1e-4)),
    (1156, torch.float64, dict(n_r=128, n_theta=256, tol=1e-4, pad=4))])
def test_noalloc_takes_plans_near_the_scratch_size(n, dtype, kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_2014_amd as ps
    from paper_1409_2014_amd import _binding as B
    print(f"case: phi_solve_noalloc near the scratch size N={n} {dtype}", flush=True)
    plan = ps.Plan(n, 16.0 / n, dtype=dtype, **kw)
    rho = torch.rand((n, n), dtype=dtype, device="cuda", generator=torch.Generator(device="cuda").manual_seed(n))
    want, got = plan.solve(rho), torch.empty_like(rho)
    st = B.lib().phi_solve_noalloc(plan._handle, ctypes.c_void_p(rho.data_ptr()), ctypes.c_void_p(got.data_ptr()),
                                   ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    B.check(st, plan._handle)
    torch.cuda.synchronize()
    plan.close()
    assert torch.equal(got, want)
