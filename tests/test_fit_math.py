"""The helix step's path and Jacobian (tpc_fit_math.hpp, compiled for the
host) against the same in extended precision, over all turns: series near
zero, half angles beyond, a few units of rounding everywhere.

Tolerances, in the entry's own scale: 8 units of rounding for the path (its
chain is about five operations long), 128 for the Jacobian, whose entries
divide by the cosines (0.43 at the largest |sin phi| here) up to three times;
the series' remainders (7e-14 of a term of at most 0.017) lie below."""
import os
import subprocess

import pytest

from paper_2412_13755_amd import build

SRC = r"""
#include <cmath>
#include <cstdio>
#include <random>
#include "tpc_fit_math.hpp"
typedef long double L;
static L coef[31];
// (f02, f04, f12, path, f14, y, z) of a step, by the chord and its half angle
static void exact(L s, L t, L w, L d, L kb, L *o) {
    const L kap = kb * w, s2 = s + kap * d, c = sqrtl((1 - s) * (1 + s)), c2 = sqrtl((1 - s2) * (1 + s2)), den = c + c2;
    const L T = (s + s2) / den, sq = sqrtl(1 + T * T), ch = fabsl(d) * sq, u = kap * ch / 2, sg = d >= 0 ? 1 : -1;
    L g = 0, gd = 0;
    if (fabsl(u) < 0.35L) {
        for (int q = 30; q >= 0; --q) g = g * u * u + coef[q];
        for (int q = 30; q >= 1; --q) gd = gd * u * u + 2 * q * coef[q];
        gd *= u;
    } else {
        g = asinl(u) / u;
        gd = (1 / sqrtl((1 - u) * (1 + u)) - g) / u;
    }
    const L arc = sg * ch * g, Ts = (2 + T * (s / c + s2 / c2)) / den, Tk = d * (1 + T * s2 / c2) / den;
    const L cT = fabsl(d) * T / (sq * sqrtl((1 - u) * (1 + u)));
    o[0] = d * Ts;
    o[1] = d * kb * Tk;
    o[2] = t * sg * cT * Ts;
    o[3] = arc;
    o[4] = t * kb * sg * (ch * ch / 2 * gd + cT * Tk);
    o[5] = d * T;
    o[6] = t * arc;
}
int main() {
    for (int q = 0; q <= 30; ++q) {
        L a = 1;
        for (int j = 1; j <= q; ++j) a *= (L)(2 * j - 1) / (2 * j);
        coef[q] = a / (2 * q + 1);
    }
    std::mt19937_64 r(5);
    std::uniform_real_distribution<double> U(0, 1);
    const double kb = -0.00299792458 * 0.5, edge[] = {0.001, 0.025, 0.05, 0.1, 0.3, 0.6, 3.0};
    double worst[7][7] = {};
    for (int i = 0; i < 400000; ++i) {
        const double s = (U(r) < 0.5 ? 0.3 : 0.9) * (2 * U(r) - 1), d = U(r) < 0.8 ? -1.0596 : U(r) * 8 - 4;
        const double kd = pow(10, -5 + 5.25 * U(r)) * (U(r) < 0.5 ? 1 : -1), t = 2 * U(r) - 1, w = kd / d / kb;
        if (!(fabs(s + kd) < 0.9)) continue;
        double p[5] = {0, 0, s, t, w};
        StepJac J;
        if (!helix_step<double, double>(p, d, kb, 0.999f, J)) return 1;
        L o[7];
        exact(s, t, w, d, kb, o);
        const L turn = fabsl(asinl((L)s + (L)kb * w * d) - asinl((L)s));
        int b = 0;
        while (b < 6 && turn >= edge[b]) ++b;
        const double got[7] = {J.f02, J.f04, J.f12, J.f13, J.f14, p[0], p[1]};
        const L at = fabsl((L)t), sc[7] = {fabsl(o[0]), fabsl(o[1]), fabsl((L)d) * at, fabsl(o[3]),
                                           at * fabsl((L)kb) * d * d, fabsl((L)d), fabsl(o[6])};
        for (int q = 0; q < 7; ++q) worst[b][q] = fmax(worst[b][q], (double)(fabsl(got[q] - o[q]) / sc[q]));
    }
    for (int b = 0; b < 7; ++b) {
        printf("%g", edge[b]);
        for (int q = 0; q < 7; ++q) printf(" %.3g", worst[b][q]);
        printf("\n");
    }
    return 0;
}
"""

EPS = 2.0 ** -52
NAMES = ("f02", "f04", "f12", "path", "f14", "y", "z")
TOL = dict(f02=128 * EPS, f04=128 * EPS, f12=128 * EPS, path=8 * EPS, f14=128 * EPS, y=128 * EPS, z=8 * EPS)


def test_step_over_all_turns(tmp_path):
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not found")
    src, exe = tmp_path / "step.hip", tmp_path / "step"
    src.write_text(SRC)
    subprocess.run([hipcc, "-O2", "-std=c++17", "--offload-host-only", "-I", build.CSRC, str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    rows = [line.split() for line in out.splitlines()]
    assert len(rows) == 7
    bad = [(r[0], n, v) for r in rows for n, v in zip(NAMES, r[1:]) if not float(v) <= TOL[n]]
    print(out)
    assert not bad, "errors (turns below, entry, error): %r" % bad
