"""phi_solve_timed runs the layout of the eager solve it measures: its kernels are on
as many streams, read off a profile of both calls.  One plan per layout: one launch
for both branches, separate launches on one stream, and two streams by size and by
flag; forward and transposed."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def streams_of(call):
    """Number of streams that the kernels of four such calls run on (the profiler may
    miss an event of a call, so no single one is counted on)."""
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        for _ in range(4):
            call()
        torch.cuda.synchronize()
    events = [e for e in prof.events() if e.device_type == torch.autograd.DeviceType.CUDA and "phi::" in e.name]
    assert len(events) >= 12
    return len({e.device_resource_id for e in events})


@pytest.mark.parametrize("n,dtype,kw,streams", [
    (64, torch.float64, {}, 1), (1024, torch.float64, {}, 1), (600, torch.float64, {}, 1),
    (1024, torch.float64, {"two_streams": True}, 2), (2048, torch.float32, {}, 2)])
def test_timed_solve_runs_the_eager_layout(n, dtype, kw, streams):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_2014_amd as ps
    print(f"case: layout of a timed solve N={n} {dtype} {kw}", flush=True)
    plan = ps.Plan(n, 16.0 / n, dtype=dtype, **kw)
    rho = torch.rand((n, n), dtype=dtype, device="cuda", generator=torch.Generator(device="cuda").manual_seed(n))
    out = torch.empty_like(rho)
    for adjoint in (False, True):
        eager = streams_of(lambda: (plan.solve_adjoint if adjoint else plan.solve)(rho, out))
        want = out.clone()
        timed = streams_of(lambda: plan.solve_timed(rho, out, adjoint=adjoint))
        print(f"  adjoint {adjoint}: eager on {eager} stream(s), timed on {timed}", flush=True)
        assert eager == streams and timed == streams
        assert torch.equal(out, want)
    plan.close()
