"""What the ratios of a clip search allow (csrc/clip_grid.h), compiled on its own: the common fraction that the one-pass search
needs is found where it exists and only there, never for ratios that are equal, and the signs of a lone value that leaves the
ratio open are those for which the quantiser's errors say so."""
import os
import subprocess
from fractions import Fraction

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_05413_amd", "csrc")
PROGRAM = r"""
#include "clip_grid.h"
#include <cstdio>
int main()
{
    int n, K;
    double lo;
    while (std::scanf("%d %lf %d", &n, &lo, &K) == 3) {
        float grid[sr::kMaxClipGrid];
        for (int i = 0; i < n; ++i) grid[i] = (float)(1.0 - (1.0 - (double)(float)lo) * (double)i / (double)(n - 1));
        std::printf("%d %d\n", sr::clip_grid_denominator(grid, n), sr::undecided_signs(grid, n, K));
    }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    (d / "grid.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, "-o", str(d / "grid"), str(d / "grid.cpp")], check=True)

    def run(cases):
        text = "".join("%d %.17g %d\n" % c for c in cases)
        out = subprocess.run([str(d / "grid")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, l.split())) for l in out.splitlines()]
    return run


def test_common_fraction(ask):
    cases = [(n, p / 200, 4096) for n in (2, 3, 5, 6, 11, 21, 26, 32) for p in (1, 25, 50, 74, 99, 100, 101, 138, 150, 160, 180, 199)]
    for (n, lo, _), (q, _) in zip(cases, ask(cases)):
        step = (1 - Fraction(lo).limit_denominator(200)) / (n - 1)
        exact = step.denominator if (1 - step * (n - 1)).denominator <= step.denominator else None
        assert q == (exact if exact is not None and exact <= 100 else 0), (n, lo, q, exact)


@pytest.mark.parametrize("lo", [1.0, 1 - 2 ** -24, 1 - 2 ** -22])
def test_equal_ratios_have_none(ask, lo):
    assert [q for q, _ in ask([(n, lo, 4096) for n in (2, 5, 21, 32)])] == [0] * 4


def test_signs_of_a_lone_value(ask):
    cases = [(n, lo, K) for n, lo in ((2, 0.5), (2, 0.9), (11, 0.5), (21, 0.5), (21, 0.8), (26, 0.5), (32, 0.69)) for K in (2048, 4096, 8192, 14336, 28672)]
    seen = set()
    for (n, lo, K), (_, signs) in zip(cases, ask(cases)):
        d = np.linspace(1.0, lo, n) / 7
        want = 0
        for bit, y in ((1, 1.0), (2, -1.0)):
            e = (y - d * np.clip(np.rint(y / d), -8, 7)) ** 2
            margin = np.sort(e)[1] - e.min()
            if abs(margin - K * 2.0 ** -16 / 196) < 1e-7:         # on the line: either answer
                want |= signs & bit
            elif margin < K * 2.0 ** -16 / 196:
                want |= bit
        assert signs == want, (n, lo, K, signs, want)
        seen.add(signs)
    assert seen == {0, 2, 3}
