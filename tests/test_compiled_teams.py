"""The teams that the library compiles, as its own headers give them (CPU).

A host-only compile of the headers prints every team that a kernel is instantiated
with: line length, threads, radix plan, slots.  The transform is then run in numpy
with the index formulas of TeamFFT (csrc/psn_device.h): each stage must write every
position once, the result must be the DFT (log2 n stages of rounding, below 1e-13
of the largest output), and the positions that a forward transform leaves in each
thread and slot must be those that the transform with the radices reversed starts
from, over all threads and slots."""
import json
import math
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1612_01799_amd", "csrc")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

PROGRAM = r"""
#include "psn_passes.h"
#include "psn_general.h"
#include <cstdio>
using namespace psn;
template <int N, int T, class Real>
void team(const char* where) {
    using F = TeamFFT<N, T, Real, -1, false>;
    using G = TeamFFT<N, T, Real, +1, true>;
    static_assert(F::EI == G::EO && F::EO == G::EI && F::EM == G::EM, "");
    std::printf("{\"where\": \"%s\", \"n\": %d, \"T\": %d, \"bytes\": %d, \"EI\": %d, \"EO\": %d, \"EM\": %d, \"plan\": [", where, N, T,
                int(sizeof(Real)), F::EI, F::EO, F::EM);
    for (int i = 0; i < F::S; ++i) std::printf(i ? ", %d" : "%d", F::radix(i));
    std::printf("]}\n");
}
template <int N, int DT, int I>
void strided() {
    using Real = typename Prec<DT>::Real;
    team<N, Sched<N, DT>::v24[I].TT, Real>("axis 1");
    if constexpr (PairW2<N, DT>::value) team<N / 2, SchedP<N, DT>::v3[I].TT, Real>("axis 0, half lines");
    else team<N, Sched<N, DT>::v3[I].TT, Real>("axis 0");
}
template <int N, int DT>
void cube() {
    using Real = typename Prec<DT>::Real;
    team<N, Cfg<N, DT>::T, Real>("axis 2");
    if constexpr (PlaneCfg<N, DT>::value) {
        team<N, PlaneCfg<N, DT>::T, Real>("plane");
    } else {
        strided<N, DT, 0>();
        strided<N, DT, 1>();
        strided<N, DT, 2>();
        strided<N, DT, 3>();
    }
}
template <int N, class Real>
void grid() {
    team<N, GCfg<2 * N, Real, 1>::T, Real>("grid axis 2");
    team<N, GCfg<2 * N, Real, 2>::T, Real>("grid axis 1");
    if constexpr (wide_lines<Real>(N) != 0) team<N, GCfg<2 * N, Real, 3>::T, Real>("grid axis 0");
    if constexpr (wide_lines<Real>(N) >= 0) team<N, GCfg<2 * N, Real, 3, true>::T, Real>("grid axis 0");
}
int main() {
#define TEAMS(N) cube<N, DT_F64>(), cube<N, DT_F32>(), cube<N, DT_SPLIT>(), grid<N, float>(), grid<N, double>();
    PSN_FOR_EACH_SIZE(TEAMS)
}
"""


@pytest.fixture(scope="module")
def teams(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc is not here")
    d = tmp_path_factory.mktemp("teams")
    src, exe = d / "teams.hip", d / "teams"
    src.write_text(PROGRAM)
    r = subprocess.run([HIPCC, "--cuda-host-only", "-std=c++17", "-O0", "-w", "-I", CSRC, "-x", "hip", str(src), "-o",
                        str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0
    return [json.loads(line) for line in out.stdout.splitlines()]


def _held(n, T, r):
    """(thread, round, first position) of each butterfly of radix r: TeamFFT::has."""
    nb = n // r
    return [(t, s, t + T * s) for s in range(-(-nb // T)) for t in range(T) if t + T * s < nb]


def _run(x, T, sign, plan):
    n = len(x)
    tw = np.exp(-2j * np.pi * np.arange(2 * n) / (2 * n))
    lds, ns = np.array(x, complex), 1
    for i, r in enumerate(plan):
        out = np.full(n, np.nan, complex)
        m = np.arange(r)
        dft = np.exp(sign * 2j * np.pi * np.outer(m, m) / r)
        for _, _, b in _held(n, T, r):
            w = tw[m * (b % ns) * (2 * n // (ns * r))]
            v = dft @ (lds[b + m * (n // r)] * (w if sign < 0 else np.conj(w)))
            pos = b + m * (n // r) if i == len(plan) - 1 else (b // ns) * ns * r + b % ns + m * ns
            assert np.isnan(out[pos]).all(), "written twice"
            out[pos] = v
        assert not np.isnan(out).any(), "a hole"
        lds, ns = out, ns * r
    return lds


def _in_pos(n, T, plan):
    r0 = plan[0]
    return {(t, s * r0 + j): t + T * s + j * (n // r0) for t, s, _ in _held(n, T, r0) for j in range(r0)}


def _out_pos(n, T, plan):
    rl, nb = plan[-1], n // plan[-1]
    pos = {}
    for t in range(T):
        for e in range(-(-nb // T) * rl):
            if t + T * (e // rl) < nb:   # the round holds a butterfly of this thread
                pos[t, e] = t + T * (e // rl) + (e % rl) * nb
    return pos


def test_every_team_is_the_dft(teams):
    lines = {(c["n"], c["T"], tuple(c["plan"])) for c in teams}
    assert {n for n, _, _ in lines} >= {8, 12, 48, 96, 162, 384, 512}
    for n, T, plan in sorted(lines):
        assert math.prod(plan) == n
        rng = np.random.default_rng(n)
        x = rng.standard_normal(n) + 1j * rng.standard_normal(n)
        for p in (list(plan), list(plan)[::-1]):
            for sign, ref in ((-1, np.fft.fft(x)), (1, np.fft.ifft(x) * n)):
                assert np.abs(_run(x, T, sign, p) - ref).max() <= 1e-13 * np.abs(ref).max(), (n, T, p)


def test_forward_output_is_where_the_reversed_transform_starts(teams):
    for n, T, plan in sorted({(c["n"], c["T"], tuple(c["plan"])) for c in teams}):
        out = _out_pos(n, T, list(plan))
        assert sorted(out.values()) == list(range(n))
        assert out == _in_pos(n, T, list(plan)[::-1]), (n, T, plan)


def test_slots_and_teams_by_the_rules(teams):
    for c in teams:
        n, T, plan = c["n"], c["T"], c["plan"]
        slots = [-(-(n // r) // T) * r for r in plan]
        assert (c["EI"], c["EO"], c["EM"]) == (slots[0], slots[-1], max(slots)), c
        if "axis 2" in c["where"]:
            assert c["EI"] == c["EO"] == n // T, c   # the contiguous passes have no idle lane
        if n >= 48 and n & (n - 1) and n // T not in (12, 20):
            assert plan[0] in (8, 9) and len(plan) == 3, c


def test_a_wrong_reversed_layout_is_seen(teams):
    c = next(c for c in teams if c["n"] == 160 and c["T"] == 32)
    n, T, plan = c["n"], c["T"], c["plan"]
    assert plan[0] != plan[-1]
    assert _out_pos(n, T, plan) != _in_pos(n, T, plan)
