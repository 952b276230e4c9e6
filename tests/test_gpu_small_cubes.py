"""Cubes of n <= 64: axes 1 and 0 of a k2 plane in one workgroup.

White noise excites every frequency, with the packed column (k2 = 0 and n) and
its self-conjugate rows; an anisotropic box makes the three axes' spectra
differ, so that exchanged axes would show.  In place and out of place must
agree bitwise, and so must a batch that takes more than one launch table."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_common import TOL, max_rel, torch_cuda

pytestmark = pytest.mark.gpu
psn = pytest.importorskip("paper_1612_01799_amd")


@pytest.mark.parametrize("n", [8, 12, 16, 24, 32, 48, 64])
def test_plane_passes_on_white_noise(n):
    torch = torch_cuda()
    box = W.Box((-1.0, -1.3, -0.8), (1.2, 1.1, 1.5), (n, n, n))
    rho = np.random.default_rng(n).standard_normal((n, n, n))
    ref = O.solve(rho, O.half_spectrum(O.kernel_spectrum(box, 1e-12)))
    for dtype in ("f32", "f64", "split"):
        print(f"case n={n} {dtype}", flush=True)
        plan = psn.Plan(n, box=(box.a, box.b), tol=1e-12, dtype=dtype).build()
        x = torch.from_numpy(rho).to("cuda", plan.io_dtype())
        u = plan.solve(x)
        v = x.clone()
        plan.solve(v, out=v)
        torch.cuda.synchronize()
        assert torch.equal(u, v)
        assert max_rel(u.double().cpu().numpy(), ref) <= TOL[dtype], dtype


def test_more_small_cubes_than_one_launch_table():
    torch = torch_cuda()
    n, count = 12, 33
    plan = psn.Plan(n, 1.0, 1e-12, "f32").build()
    rng = np.random.default_rng(3)
    rhos = [torch.from_numpy(rng.standard_normal((n, n, n))).to("cuda", torch.float32) for _ in range(count)]
    outs = psn.solve_batched([plan] * count, rhos)
    one = [plan.solve(r) for r in rhos]
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(outs, one))
