"""Teams whose threads do not all hold the same number of butterflies (CPU).

Lines of 48 points and more with an odd factor run in three stages 8, m, g (two
for 81 points) on N / 8 threads or on the next power of two: the N / R
butterflies of a stage are dealt out in rounds of T, the last one partly
filled (csrc/psn_device.h: mid_plan, TeamFFT::has).  This restates the plan and
the positions and checks them against numpy's FFT for every line length of the
compiled sizes, their halves (the four half-length chains) and both orders of
the radices.  Each stage must write every position once, the forward output
layout must be the reversed transform's input layout, and the result must be
the DFT to FP64 rounding (log2(n) stages times a few 2^-53 of the largest
output, below 1e-13)."""
import math

import numpy as np
import pytest

SIZES = [48, 96, 160, 162, 192, 320, 384]
LINES = sorted(set(SIZES + [h for n in SIZES if n >= 96 for h in [n // 2]]))


def mid_plan(n):
    first = 8 if n % 8 == 0 else 9
    rem = n // first
    last = first
    while rem % last:
        last = last // 2 if first == 8 else last // 3
    mid = rem // last
    return [first, last] if mid == 1 else [first, mid, last]


def teams(n):
    e = 8 if n % 8 == 0 else 9
    t = n // e
    p = 1
    while p < t:
        p *= 2
    return sorted({t, p if n % 8 == 0 else t})


def slots(n, T, r):
    """(thread, slot, first position) of each element of a stage of radix r: slot s r + j holds position b + j n / r."""
    nb = n // r
    return [(t, s, t + T * s) for s in range(-(-nb // T)) for t in range(T) if t + T * s < nb]


def run(x, n, T, sign, plan):
    tw = np.exp(-2j * np.pi * np.arange(2 * n) / (2 * n))
    lds, ns = np.array(x, complex), 1
    for i, r in enumerate(plan):
        out = np.full(n, np.nan, complex)
        m = np.arange(r)
        dft = np.exp(sign * 2j * np.pi * np.outer(m, m) / r)
        for _, _, b in slots(n, T, r):
            v = lds[b + m * (n // r)]
            w = tw[m * (b % ns) * (2 * n // (ns * r))]
            v = dft @ (v * (w if sign < 0 else np.conj(w)))
            # the last stage leaves slot j at b + j n / r; the others write to LDS
            pos = b + m * (n // r) if i == len(plan) - 1 else (b // ns) * ns * r + b % ns + m * ns
            assert np.isnan(out[pos]).all(), "written twice"
            out[pos] = v
        assert not np.isnan(out).any(), "a hole"
        lds, ns = out, ns * r
    return lds


@pytest.mark.parametrize("n", [n for n in LINES if n % 2 == 0 or n == 81])
def test_uneven_teams_are_the_dft(n):
    if n < 48:
        pytest.skip("short lines keep the even plan")
    plan = mid_plan(n)
    assert math.prod(plan) == n and set(plan) <= {2, 3, 4, 5, 6, 8, 9}
    rng = np.random.default_rng(n)
    x = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    for T in teams(n):
        for p in (plan, plan[::-1]):
            f = run(x, n, T, -1, p)
            assert np.abs(f - np.fft.fft(x)).max() <= 1e-13 * np.abs(f).max()
            b = run(x, n, T, +1, p)
            assert np.abs(b - np.fft.ifft(x) * n).max() <= 1e-13 * np.abs(b).max()
        # forward out layout (last radix) = reversed transform's in layout (its first radix)
        assert slots(n, T, plan[-1]) == slots(n, T, plan[::-1][0])


def test_a_wrong_round_stride_is_seen():
    n, T, plan = 160, 32, mid_plan(160)
    x = np.random.default_rng(1).standard_normal(n) + 0j
    good = run(x, n, T, -1, plan)
    tw = np.exp(-2j * np.pi * np.arange(2 * n) / (2 * n))
    # the second stage's twiddle index without its round offset T s
    lds = np.array(x, complex)
    ns = 1
    for i, r in enumerate(plan):
        out = np.zeros(n, complex)
        m = np.arange(r)
        dft = np.exp(-2j * np.pi * np.outer(m, m) / r)
        for t, s, b in slots(n, T, r):
            k = t % ns if i == 2 else b % ns
            v = dft @ (lds[b + m * (n // r)] * tw[m * k * (2 * n // (ns * r))])
            out[b + m * (n // r) if i == len(plan) - 1 else (b // ns) * ns * r + b % ns + m * ns] = v
        lds, ns = out, ns * r
    assert np.abs(lds - good).max() > 1e-3 * np.abs(good).max()
