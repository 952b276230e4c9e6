"""The strided passes' tile candidates at the sizes whose teams are uneven, or
whose W2 is paired over lanes, against the oracle; and bitwise repeatability
(a missing barrier between two rounds of a stage would show as differences)."""
import pytest

import oracle as O
import workloads as W
from gpu_common import TOL, gpu_solve, max_rel, oracle_symbol, torch_cuda

pytestmark = pytest.mark.gpu
psn = pytest.importorskip("paper_1612_01799_amd")


@pytest.mark.parametrize("n,dtype", [(96, "f64"), (128, "split"), (162, "f64"), (192, "f32"), (192, "f64"),
                                     (320, "f32"), (320, "split"), (384, "f32"), (384, "f64")])
def test_candidates_and_repeatability(n, dtype):
    torch = torch_cuda()
    print(f"case n={n} {dtype}", flush=True)
    L = 3.0
    rho = W.mixture_density(W.draw_mixture(600 + n, 5, -1.0, 1.0, 0.4, 0.65, 0.5, 1.5, W.Box.cube(L, n)))
    ref = O.solve(rho, oracle_symbol(n, L))
    plan = psn.Plan(n, L, 1e-12, dtype).build()
    x = torch.from_numpy(rho).to("cuda", plan.io_dtype())
    for v in range(4):
        plan.set_schedule(v, v)
        u = gpu_solve(psn, torch, n, L, dtype, rho, plan=plan)
        assert max_rel(u, ref) <= TOL[dtype], v
        a, b = plan.solve(x), plan.solve(x)
        torch.cuda.synchronize()
        assert torch.equal(a, b), v


@pytest.mark.parametrize("n3", [(384, 96, 160), (160, 320, 48), (162, 192, 96)])
def test_grid_steps_with_uneven_teams(n3):
    torch = torch_cuda()
    print(f"grid {n3}", flush=True)
    b = tuple(0.02 * (q - 1) for q in n3)
    box = W.Box(tuple(-v for v in b), b, n3)
    s = min(b)
    rho = W.mixture_density(W.draw_mixture(7, 4, -s / 3, s / 3, 0.2 * s, 0.3 * s, 0.5, 1.5, box))
    ref = O.solve(rho, O.half_spectrum(O.kernel_spectrum(box, 1e-12)))
    for dtype in ("f32", "f64"):
        plan = psn.Plan(n3, box=(box.a, box.b), tol=1e-12, dtype=dtype).build()
        u = plan.solve(torch.from_numpy(rho).to("cuda", plan.io_dtype()))
        torch.cuda.synchronize()
        assert max_rel(u.double().cpu().numpy(), ref) <= TOL[dtype], dtype
