"""The nonlinear substep's rotation e^{i phi} in the stepper's row passes: phases
inside the branch-free range, at its edge and beyond it (1e6; the library routine
takes those points again), forward and in the reverse pass, on sides whose row
blocks are one wave and wider, against the oracle stepper with the periodic
potential.  A phase of size M carries an error of a few M ulps from its own
products whatever the sine does, which is what the bars allow."""
import numpy as np
import pytest

from oracle import ds_stepper as D
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EPS = {torch.float64: 2.0 ** -53, torch.float32: 2.0 ** -24}
CDT = {torch.float64: torch.complex128, torch.float32: torch.complex64}


def rel_linf(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


@pytest.mark.parametrize("n,half", [(16, 3.0), (128, 6.0), (512, 6.0), (1024, 8.0)])
@pytest.mark.parametrize("dtype,phase", [(torch.float64, 0.3), (torch.float64, 400.0), (torch.float64, 9.9e5),
                                         (torch.float64, 3.0e6), (torch.float32, 0.3), (torch.float32, 60.0)])
def test_rotation_in_both_directions(n, half, dtype, phase):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_2014_amd as ps
    print(f"case: rotation N={n} {dtype} largest phase {phase}", flush=True)
    h, tau = 2 * half / n, 1e-3
    x, y, _ = W.grid_2d(n, half)
    u0 = np.exp(-(x ** 2 + 2 * y ** 2)).astype(np.complex128)      # |u|^2 <= 1: the phase's largest value is c tau
    c = phase / tau
    kw = dict(alpha=1.0, tau=tau, potential="periodic", c_local=c, c_potential=0.5 * c)
    st = ps.DSStepper(n, h, dtype=dtype, **kw)
    p = D.DSParams(n=n, h=h, **kw)
    u = torch.as_tensor(u0, dtype=CDT[dtype], device="cuda").contiguous()
    start = u.cpu().numpy().astype(np.complex128)
    # products and sums of the phase, and rounding of the density (a transform's)
    bar = EPS[dtype] * (64.0 * phase + 64.0)
    got = st.forward(u.clone(), 1).cpu().numpy()
    err = rel_linf(got, D.evolve(start, p, 1))
    _, grad, _ = st.loss_and_grad(u, 1, 1)
    _, ref = D.loss_l4_gradient(start, p, 1)
    gerr = rel_linf(grad.cpu().numpy(), ref)
    st.close()
    print(f"  forward {err:.2e} gradient {gerr:.2e} (bar {bar:.1e}, {16 * bar:.1e})", flush=True)
    assert np.all(np.isfinite(got.view(np.float64 if dtype == torch.float64 else np.float32)))
    assert err <= bar and gerr <= 16 * bar


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_a_phase_that_is_not_a_number_stays_one(dtype):
    """An infinite density makes its phase NaN; the other points are unaffected by
    the branch (the transforms spread the NaN, so the field is NaN throughout, as it
    is from the library routine)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_2014_amd as ps
    print(f"case: rotation of a NaN phase {dtype}", flush=True)
    st = ps.DSStepper(64, 0.25, dtype=dtype, tau=1e-3, potential="periodic")
    u = torch.ones((64, 64), dtype=CDT[dtype], device="cuda")
    u[3, 5] = float("inf")
    out = st.forward(u, 1)
    torch.cuda.synchronize()
    st.close()
    assert bool(torch.isnan(torch.view_as_real(out)).any())


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("phase", [0.3, 9.9e5, 1.0e6, 1.5e6, 3.1e7])
def test_rotation_of_a_constant_field(dtype, phase):
    """A constant field of size 1/2 goes through the transforms exactly (sums of equal
    values, the zero mode's factors are 1) and its periodic potential is 0, so a step
    multiplies it by e^{i phase} alone, on either side of the branch-free range (1e6)
    and at its edge.  The phase is the product of two rounded numbers; the sine and
    cosine are within 4 ulps of 1, and the products of the field add rounding."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_2014_amd as ps
    print(f"case: rotation of a constant field {dtype} phase {phase}", flush=True)
    real = np.float64 if dtype == torch.float64 else np.float32
    tau, c = 2.0 ** -10, 4.0 * phase * 2.0 ** 10       # |u|^2 = 1/4; tau and |u|^2 are exact
    st = ps.DSStepper(64, 0.25, dtype=dtype, tau=tau, potential="periodic", c_local=c, c_potential=c)
    u = torch.full((64, 64), 0.5, dtype=CDT[dtype], device="cuda")
    got = st.forward(u, 1).cpu().numpy()
    st.close()
    want = 0.5 * np.exp(1j * float(real(c) * real(0.25) * real(tau)))
    assert np.max(np.abs(got - want)) <= 8 * EPS[dtype]
