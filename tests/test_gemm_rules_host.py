"""The launch rules of the two GEMMs (csrc/gemm_rules.h), compiled on their own: what they predict is possible and grows with
the work, and what they choose is no slower than the two large tiles they started from."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_05413_amd", "csrc")
PROGRAM = r"""
#include "gemm_rules.h"
#include <cstdio>
#include <cstring>
int main()
{
    char kind[16];
    long long M, N, K;
    while (std::scanf("%15s %lld %lld %lld", kind, &M, &N, &K) == 4) {
        const bool f6 = !std::strcmp(kind, "f6");
        const sr::GemmShape s = f6 ? sr::f6_shape(M, N, K, 256) : sr::packed_shape(M, N, K, 256);
        const sr::GemmConfig *c = f6 ? sr::f6_config(s) : sr::packed_config(s);
        std::printf("%d %.6f", c->id, sr::gemm_cost(*c, s));
        if (f6) for (const sr::GemmConfig &d : sr::kF6Configs) std::printf(" %.6f", sr::gemm_cost(d, s));
        else for (const sr::GemmConfig &d : sr::kPackedConfigs) std::printf(" %.6f", sr::gemm_cost(d, s));
        std::printf("\n");
    }
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, "-o", str(d / "rules"), str(d / "rules.cpp")], check=True)

    def run(kind, shapes):
        text = "".join("%s %d %d %d\n" % (kind, *s) for s in shapes)
        out = subprocess.run([str(d / "rules")], input=text, capture_output=True, text=True, check=True).stdout
        rows = [[float(v) for v in l.split()] for l in out.splitlines()]
        return [(int(r[0]), r[1], r[2:]) for r in rows]          # choice, its time, the time of every configuration
    return run


def test_gpu_tests_force_every_configuration(rule, tmp_path):
    """A number that no rule knows would silently run the automatic choice."""
    import test_gpu_f6_configs as f6
    import test_gpu_gemm_configs as packed
    (tmp_path / "ids.cpp").write_text("""
#include "gemm_rules.h"
#include <cstdio>
int main()
{
    for (const sr::GemmConfig &c : sr::kPackedConfigs) std::printf("packed %d %d %d\\n", c.id, c.bm, c.bn);
    for (const sr::GemmConfig &c : sr::kF6Configs) std::printf("f6 %d %d %d\\n", c.id, c.bm, c.bn);
}
""")
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(tmp_path / "ids"), str(tmp_path / "ids.cpp")], check=True)
    out = subprocess.run([str(tmp_path / "ids")], capture_output=True, text=True, check=True).stdout
    for kind, module in (("packed", packed), ("f6", f6)):
        tiles = {int(i): (int(m), int(n)) for k, i, m, n in (l.split() for l in out.splitlines()) if k == kind}
        assert sorted(tiles) == sorted(module.CONFIGS)
        assert {i: t for i, t in tiles.items() if i < 1000} == module.TILES


MS = [17, 31, 64, 129, 200, 333, 513, 777, 1024, 2048, 3000, 4096, 8192, 16384, 65536]
NS = [16, 512, 1040, 2784, 4096, 6144, 14336, 28672]
KS = {"packed": [256, 512, 768, 1024, 2048, 4096, 8192, 14336, 28672], "f6": [128, 256, 512, 1024, 2048, 4096, 8192, 14336, 28672]}
OPS = {"packed": 3.7e15, "f6": 6.2e15}                           # the most the bare matrix loops reach


@pytest.mark.parametrize("kind", ["packed", "f6"])
def test_predictions_grow_with_the_work(rule, kind):
    for axis, values in enumerate((MS, NS, KS[kind])):
        shapes = [(m, n, k) for m in MS for n in NS for k in KS[kind]]
        at = dict(zip(shapes, rule(kind, shapes)))
        for s in shapes:
            i = values.index(s[axis])
            if i + 1 < len(values):
                t = list(s)
                t[axis] = values[i + 1]
                assert all(a <= b * (1 + 1e-6) for a, b in zip(at[s][2], at[tuple(t)][2])), (s, t)


@pytest.mark.parametrize("kind", ["packed", "f6"])
def test_no_prediction_beats_the_matrix_pipe(rule, kind):
    shapes = [(m, n, k) for m in MS for n in NS for k in KS[kind]]
    for s, (choice, us, every) in zip(shapes, rule(kind, shapes)):
        assert min(every) > 0 and us >= min(every)
        assert us > 2e6 * s[0] * s[1] * s[2] / OPS[kind], s


# Measured, us, weights from HBM: shape -> configuration -> time, the two large tiles and the candidates.
MEASURED = {
    "packed": {(224, 13616, 4096): {14: 22.99, 15: 26.98, 18: 26.47, 19: 25.15, 20: 20.47},
               (1937, 4640, 8192): {14: 79.79, 15: 93.75, 18: 88.70, 20: 84.59},
               (512, 4096, 14336): {14: 60.59, 15: 74.17, 17: 51.52, 19: 52.97, 20: 40.68, 64064: 37.75},
               (190, 9456, 8192): {14: 38.79, 15: 45.67, 17: 40.11, 19: 34.29, 20: 27.95, 64064: 26.17},
               (4096, 14336, 256): {14: 40.01, 15: 37.31, 17: 50.06, 18: 41.43, 19: 47.20, 20: 56.23},
               (8192, 14336, 256): {14: 74.83, 15: 70.40, 17: 99.36, 18: 77.69, 19: 94.73, 20: 109.30},
               (16384, 4096, 1024): {14: 83.17, 15: 78.29, 17: 111.15, 18: 91.37, 19: 107.38, 20: 103.50}},
    "f6": {(947, 24592, 2048): {61: 51.65, 72: 50.01, 65: 61.70, 68: 64.84, 67: 58.79},      # (45.5 and 49.0 in other runs)
           (1050, 7776, 2048): {61: 16.73, 72: 17.73, 65: 27.94, 68: 29.25, 67: 26.56},
           (1062, 8576, 128): {61: 6.94, 72: 6.93, 65: 8.70, 68: 9.12, 67: 7.54, 32064: 18.40},
           (7448, 24416, 512): {61: 111.37, 72: 148.21, 65: 165.56, 68: 142.00, 67: 160.73}},
}


@pytest.mark.parametrize("kind,shape", [(k, s) for k, v in MEASURED.items() for s in v])
def test_choice_is_no_slower_than_the_large_tiles(rule, kind, shape):
    times = MEASURED[kind][shape]
    large = min(times[i] for i in ((14, 15) if kind == "packed" else (61, 65)))
    choice = rule(kind, [shape])[0][0]
    assert times[choice] <= 1.03 * large, (choice, times)
