"""Eager solves queued one behind the other, with no wait in between, equal the same
solves under graph replay bit for bit: the eager call's fork and join (events attached
to the kernels, or none where the launches stay on one stream) order its kernels as a
graph's edges do.  One size per way a solve is queued, and a batch."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def sequence(solve, inputs, stream):
    """Each input solved right behind the one before, into buffers of its own."""
    outs = [torch.empty_like(x) for x in inputs]
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for x, o in zip(inputs, outs):
            solve(x, o)
    stream.synchronize()
    return outs


def replayed(solve, inputs):
    x, o = inputs[0].clone(), torch.empty_like(inputs[0])
    solve(x, o)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        solve(x, o)
    outs = []
    for new in inputs:
        x.copy_(new)
        graph.replay()
        torch.cuda.synchronize()
        outs.append(o.clone())
    return outs


def inputs_like(shape, dtype):
    gen = torch.Generator(device="cuda").manual_seed(3)
    return [(k + 1) * torch.rand(shape, dtype=dtype, device="cuda", generator=gen) for k in range(12)]


@pytest.mark.parametrize("n,dtype,kw", [
    (64, torch.float64, {}), (514, torch.float64, {}), (1024, torch.float64, {}),
    (1024, torch.float64, {"two_streams": True}), (128, torch.float32, {"two_streams": True}),
    (1026, torch.float32, {}), (2048, torch.float32, {}), (2048, torch.float64, {}), (2050, torch.float32, {})])
def test_queued_solves_equal_replays(n, dtype, kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_2014_amd as ps
    print(f"case: queued solves N={n} {dtype} {kw}", flush=True)
    plan = ps.Plan(n, 16.0 / n, dtype=dtype, **kw)
    inputs = inputs_like((n, n), dtype)
    want = replayed(plan.solve, inputs)
    for stream in (torch.cuda.current_stream(), torch.cuda.Stream()):
        for got, ref in zip(sequence(plan.solve, inputs, stream), want):
            assert torch.equal(got, ref)
    plan.close()


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_queued_batches_equal_replays(dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_2014_amd as ps
    print(f"case: queued batches {dtype}", flush=True)
    plan = ps.BatchPlan([dict(n=n, h=16.0 / n) for n in (128, 700, 90, 512)], dtype=dtype)
    inputs = inputs_like((plan.total,), dtype)
    want = replayed(plan.solve, inputs)
    for got, ref in zip(sequence(plan.solve, inputs, torch.cuda.Stream()), want):
        assert torch.equal(got, ref)
    plan.close()


@pytest.mark.parametrize("n,dtype", [(64, torch.float64), (1024, torch.float64), (2048, torch.float32),
                                     (2050, torch.float32)])
def test_queued_transposed_solves_equal_replays(n, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_2014_amd as ps
    print(f"case: queued transposed solves N={n} {dtype}", flush=True)
    plan = ps.Plan(n, 16.0 / n, dtype=dtype)
    inputs = inputs_like((n, n), dtype)
    want = replayed(plan.solve_adjoint, inputs)
    for got, ref in zip(sequence(plan.solve_adjoint, inputs, torch.cuda.Stream()), want):
        assert torch.equal(got, ref)
    plan.close()
