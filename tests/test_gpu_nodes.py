"""The node stage of a solve (half-plane nodes; matrix instructions where the
spread tile fits 16 x 16 window cells, the general kernel beyond) against the
oracle's direct nonuniform sums, at the edges of both: one to many nodes per
group of 16, tiles of 6 to 16 cells and the first one past 16, windows smaller
than the fine grid and windows that are the whole of it (taps wrap), grids from
8 points a side, and subproblem sizes below a group."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (n, half, n_r, n_theta, tol, kwargs): kernel width w = ceil(log10 1/tol) + 1,
# tile side bin + w - 1
CASES = [
    (8, 4.0, 1, 2, 1e-12, {}),                    # one node, fine grid of 16: the window wraps
    (8, 4.0, 6, 10, 1e-12, {}),
    (16, 4.0, 5, 6, 1e-12, {}),
    (32, 4.0, 17, 34, 1e-2, {}),                  # w = 3, tile 6
    (64, 8.0, 32, 64, 1e-12, {}),                 # w = 13: tile 16, the largest on matrix instructions
    (64, 8.0, 32, 64, 1e-13, {}),                 # w = 14: tile 17, the general kernel
    (64, 8.0, 60, 60, 1e-9, {"sub_nodes": 8}),    # half a group per subproblem
    (96, 4.0, 33, 50, 1e-8, {"sub_nodes": 24}),   # a group and a half
    (100, 6.0, 16, 30, 1e-7, {"bin": 8}),         # w = 8: tile 15
    (100, 6.0, 16, 30, 1e-9, {"bin": 8}),         # w = 10: tile 17
    (128, 8.0, 24, 48, 1e-6, {"bin": 16}),
    (64, 8.0, 40, 40, 1e-6, {"kernel": "gaussian"}),   # w = 14 at tile 17
]


@pytest.mark.parametrize("n,half,n_r,n_theta,tol,kw", CASES)
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_low_frequency_part_against_direct_sums(n, half, n_r, n_theta, tol, kw, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_2014_amd as ps
    if dtype == torch.float32 and tol < 1e-7:
        tol = 1e-7
    h = 2 * half / n
    print(f"case: node stage N={n} nodes={n_r}x{n_theta} tol={tol} {kw} {dtype}", flush=True)
    rho = np.random.default_rng(n + n_r).standard_normal((n, n))
    r = torch.as_tensor(rho, dtype=dtype, device="cuda")
    plan = ps.Plan(n, h, dtype=dtype, n_r=n_r, n_theta=n_theta, tol=tol, **kw)
    got = plan.lowfreq(r).double().cpu().numpy()
    fine = plan.info["n_fine"]
    whole = plan.info["patch"] == fine
    plan.close()
    p = O.SplitParams(n=n, h=h, n_r=n_r, n_theta=n_theta, pad_side=fine)
    ref = O.i2_direct(r.double().cpu().numpy(), p)
    ref = np.real(ref[0] if isinstance(ref, tuple) else ref)
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    # two transforms, each to tol (10 tol is the stages' documented bar), and
    # their rounding
    bar = 20 * tol + (2e-6 if dtype == torch.float32 else 1e-12)
    print(f"  rel l2 {err:.3e} (bar {bar:.1e}, whole window {whole})", flush=True)
    assert err <= bar
