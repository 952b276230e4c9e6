"""White noise through the passes of n >= 96 and through the per-axis grids.

A resolved density is zero to rounding at the high frequencies, so it does not
see the packed k2 = n plane of column 0, the folded kernel indices beside n or the
ends of the spectrum.  White noise excites every frequency alike: a wrong plane of
n^2 frequencies changes u by about 0.5 / n of its largest value and a wrong line of
n by about 0.2 n^-1.5 (2e-5 at n = 512), above every tolerance here.  The boxes are
anisotropic, so that exchanged axes show."""
import functools

import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_common import TOL, max_rel, torch_cuda

pytestmark = pytest.mark.gpu
psn = pytest.importorskip("paper_1612_01799_amd")


def _box(n3, long_axis=1):
    h = (0.021 * long_axis, 0.025, 0.019)
    b = tuple(0.5 * h[q] * (n3[q] - 1) for q in range(3))
    return W.Box(tuple(-0.9 * v for v in b), b, n3)


@functools.lru_cache(maxsize=1)
def _case(n3, long_axis=1):
    rho = np.random.default_rng(sum(n3)).standard_normal(n3)
    return rho, O.solve(rho, O.half_spectrum(O.kernel_spectrum(_box(n3, long_axis), 1e-12)))


@pytest.mark.parametrize("n", [96, 128, 160, 162, 192, 256, 320, 384, 512])
def test_every_candidate(n):
    torch = torch_cuda()
    rho, ref = _case((n, n, n))
    box = _box((n, n, n))
    for dtype in ("f32", "f64", "split"):
        plan = psn.Plan(n, box=(box.a, box.b), tol=1e-12, dtype=dtype).build()
        x = torch.from_numpy(rho).to("cuda", plan.io_dtype())
        for v in range(4):
            print(f"case n={n} {dtype} candidate {v}", flush=True)
            plan.set_schedule(v, v)
            u, w = plan.solve(x), plan.solve(x)
            torch.cuda.synchronize()
            assert torch.equal(u, w), (dtype, v)
            assert max_rel(u.double().cpu().numpy(), ref) <= TOL[dtype], (dtype, v)


@pytest.mark.parametrize("n", [96, 162, 192])
def test_batch(n):
    """Several problems a launch: the column-0 workgroups of each come first."""
    torch = torch_cuda()
    rho, ref = _case((n, n, n))
    box = _box((n, n, n))
    for dtype in ("f32", "f64", "split"):
        print(f"case n={n} {dtype} batch of 5", flush=True)
        plan = psn.Plan(n, box=(box.a, box.b), tol=1e-12, dtype=dtype).build()
        x = torch.from_numpy(rho).to("cuda", plan.io_dtype())
        zero = torch.zeros_like(x)
        outs = psn.solve_batched([plan] * 5, [x, zero, x, -x, x])
        torch.cuda.synchronize()
        for i, f in enumerate((1, 0, 1, -1, 1)):
            assert np.abs(outs[i].double().cpu().numpy() - f * ref).max() <= TOL[dtype] * np.abs(ref).max(), (dtype, i)


@pytest.mark.parametrize("n3", [(96, 162, 48), (162, 48, 96), (48, 96, 162), (192, 32, 160), (160, 192, 24),
                                (384, 24, 48), (48, 320, 96), (512, 16, 64), (64, 128, 192),
                                # either side of the lines from which the axis-0 step holds 12 elements per thread
                                (96, 192, 128), (96, 256, 256), (192, 96, 192), (192, 192, 128), (192, 256, 128)])
def test_grid(n3):
    torch = torch_cuda()
    rho, ref = _case(n3)
    box = _box(n3)
    for dtype in ("f32", "f64"):
        print(f"grid {n3} {dtype}", flush=True)
        plan = psn.Plan(n3, box=(box.a, box.b), tol=1e-12, dtype=dtype).build()
        u = plan.solve(torch.from_numpy(rho).to("cuda", plan.io_dtype()))
        torch.cuda.synchronize()
        assert max_rel(u.double().cpu().numpy(), ref) <= TOL[dtype], dtype


@pytest.mark.parametrize("n", [12, 32, 96, 128, 162])
def test_fourier_correction(n):
    """The weight that the device gives the correction's symbol.  In a long box the
    near-zone radius, set by the longest side, is no longer small against the
    spacing, and the other form of the correction is another result."""
    torch = torch_cuda()
    print(f"case n={n} fourier", flush=True)
    rho, folded = _case((n, n, n), 30)
    box = _box((n, n, n), 30)
    ref = O.solve_paper_form(rho, box, 1e-12)
    assert max_rel(folded, ref) > 100 * TOL["f64"]
    plan = psn.Plan(n, box=(box.a, box.b), tol=1e-12, dtype="f64", correction="fourier").build()
    u = plan.solve(torch.from_numpy(rho).to("cuda"))
    torch.cuda.synchronize()
    assert max_rel(u.cpu().numpy(), ref) <= TOL["f64"]
