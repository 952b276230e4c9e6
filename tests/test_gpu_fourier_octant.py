"""The octant that a plan with the Fourier-series correction gives is the G-tensor
in the plan's own precision.

K also holds the correction's symbol times 8 at the all-even frequencies.  In a
long thin box the near-zone radius (set by the longest side) exceeds the spacing
of the short ones and the symbol is many times the G-tensor there, so an octant
taken as the FP32 sum less the symbol keeps the rounding of the sum.  The F32
plan's octant must be the F64 plan's rounded once (2^-24 of each value; the
slack is for values beside a tie)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_common import torch_cuda

pytestmark = pytest.mark.gpu
psn = pytest.importorskip("paper_1612_01799_amd")

BOX = W.Box((-100.0, -1.0, -1.2), (100.0, 1.0, 1.1), (16, 16, 16))


@pytest.mark.parametrize("n", [16, 96])
def test_f32_octant_is_the_f64_one_rounded_once(n):
    torch_cuda()
    print(f"case n={n}", flush=True)
    octant = {dt: psn.Plan(n, box=(BOX.a, BOX.b), tol=1e-12, dtype=dt, correction="fourier").build().kernel_octant()
              for dt in ("f32", "f64")}
    ref = octant["f64"][:, :, 1:n]   # k2 = 0 and n are stored as half sum and half difference
    assert np.all(np.abs(octant["f32"][:, :, 1:n] - ref) <= 2.0 ** -24 * (1 + 1e-6) * np.abs(ref))


def test_octant_is_the_g_tensor_where_the_symbol_is_larger():
    torch_cuda()
    ks = O.kernel_spectrum(BOX, 1e-12, with_correction=False)
    k = psn.Plan(16, box=(BOX.a, BOX.b), tol=1e-12, dtype="f64", correction="fourier").build().kernel_octant()
    assert np.max(np.abs(k - ks.octant)) <= 1e-13 * abs(ks.octant[0, 0, 0])
