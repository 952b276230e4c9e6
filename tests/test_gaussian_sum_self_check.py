"""The reported fit error of the Gaussian sum is the maximum over all its radii.

Plan creation screens the radii by interpolation and sums only those that can
hold the maximum; here every radius is summed.  Both sums carry a rounding
error of at most (5/hs + 16) u each (u = 2^-53).
"""
import numpy as np
import pytest

import paper_1612_01799_amd as psn

POINTS = 32768


@pytest.mark.parametrize("tol", [1e-4, 1e-8, 1e-12, 1e-13, 1e-14])
@pytest.mark.parametrize("n,L", [(8, 0.01), (32, 6.0), (162, 40.0)])
def test_fit_error_is_the_maximum_over_all_radii(n, L, tol):
    p = psn.Plan(n, L, tol, "f64")
    info = p.info()
    tau, w = p.gs_table()
    a, b = np.log(info["delta"]), np.log(info["R"])
    r = np.exp(a + (b - a) * np.arange(POINTS) / (POINTS - 1))
    s = np.zeros(POINTS)
    for t, c in zip(tau, w):
        s += c * np.exp(-(t * r) ** 2)
    worst = np.max(np.abs(4.0 * np.pi * r * s - 1.0))
    assert abs(info["eps_achieved"] - worst) <= 2 * (5.0 / info["hs"] + 16.0) * 2.0 ** -53
    assert info["eps_achieved"] <= tol
