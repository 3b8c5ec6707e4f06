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


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_batch_plans_hold_no_tables_of_the_stage_entry_points(dtype):
    """A batch takes solves only, so next to a single plan of the same problem it
    lacks at least the taps of the full node set (2 w values per node); its work
    lists and member views are under 64 KiB here."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_2014_amd as ps
    print(f"case: batch plan memory {dtype}", flush=True)
    member = dict(n=256, h=1.0 / 16, n_r=128, n_theta=256)
    plan, batch = ps.Plan(**member, dtype=dtype), ps.BatchPlan([member], dtype=dtype)
    taps = plan.info["n_nodes"] * 2 * plan.info["kernel_width"] * (4 if dtype == torch.float32 else 8)
    sizes = plan.info["device_bytes"], batch.device_bytes
    rho = torch.rand((256, 256), dtype=dtype, device="cuda")
    assert torch.equal(batch.solve(rho.reshape(-1)).view(256, 256), plan.solve(rho))
    plan.close()
    batch.close()
    assert sizes[1] <= sizes[0] - taps + 65536, sizes
