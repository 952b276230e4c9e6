"""The Fourier-series correction as a term of the padded kernel spectrum (CPU).

The length-n transform of an axis is the even outputs of the zero-padded
length-2n one, so C0 rho + (C2/6) Laplace_n(rho) is the padded convolution with
8 times the symbol on the all-even frequencies.  The library builds its
spectrum so; here the same sum in numpy must equal the oracle's separate
n-point transform pair.  White noise excites every frequency; both sides are
sums of O(1) terms in FP64, so they may differ by transform rounding only
(log2 of the 2^15 points times 2^-53, times 10)."""
import math

import numpy as np
import pytest

import oracle as O
import workloads as W
from oracle.correction import correction


@pytest.mark.parametrize("n", [(8, 8, 8), (12, 12, 12), (16, 16, 16)])
def test_symbol_on_even_frequencies_is_the_n_point_correction(n):
    box = W.Box((-3.0, -2.0, -1.0), (2.0, 3.5, 5.0), n)
    rho = np.random.default_rng(n[0]).standard_normal(n)
    ks = O.kernel_spectrum(box, 1e-12, with_correction=False)
    C0, C2 = correction(ks.tau, ks.w, ks.geom.delta)
    k = np.arange(n[0] + 1)
    kap = [2 * math.pi * k / ks.geom.P[q] for q in range(3)]
    sym = C0 - (C2 / 6) * (kap[0][:, None, None] ** 2 + kap[1][None, :, None] ** 2 + kap[2][None, None, :] ** 2)
    even = (k[:, None, None] | k[None, :, None] | k[None, None, :]) % 2 == 0
    tol = 10 * 15 * 2.0 ** -53
    ref = O.solve_paper_form(rho, box, 1e-12)
    scale = np.abs(ref).max()
    G = ks.octant
    ks.octant = G + 8 * sym * even
    assert np.abs(O.solve(rho, O.half_spectrum(ks)) - ref).max() <= tol * scale
    # the symbol on every frequency (the folded form) is another result for such a density
    ks.octant = G + sym
    assert np.abs(O.solve(rho, O.half_spectrum(ks)) - ref).max() > 100 * tol * scale
