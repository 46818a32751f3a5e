"""Which workgroup takes which tile (csrc/gemm_rules.h), compiled on its own: every tile of a grid exactly once, whatever the
grid's shape, the split over the XCDs and the number of workgroups; and no valid tile behind an invalid one."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_05413_amd", "csrc")
PROGRAM = r"""
#include "gemm_rules.h"
#include <cstdio>
#include <initializer_list>
#include <vector>
int main()
{
    long checked = 0;
    for (int tm = 1; tm <= 41; ++tm)
        for (int tn = 1; tn <= 61; tn += tm > 20 ? 3 : 1)
            for (int split : {sr::choose_xcd_split(tm, tn, 256, 128), sr::kXcdRuns, 0})
                for (int most : {8, 16, 248, 252, 256, 512}) {
                    if (split > 0 && most % 8) continue;             // rectangles are asked for with multiples of 8 only
                    const int grid = (int)sr::tile_workgroups(most, (long)tm * tn, split);
                    std::vector<int> seen(tm * tn, 0);
                    for (int v0 = 0; v0 < grid; ++v0) {
                        int m = -1, n = -1, v = v0;
                        for (; sr::tile_exists(v, tm, tn, split); v += grid) {
                            sr::tile_origin(v, tm, tn, split, 256, 128, m, n);
                            if (m % 256 || n % 128 || m / 256 >= tm || n / 128 >= tn || m < 0 || n < 0) return std::printf("outside %d %d %d %d\n", tm, tn, split, v), 1;
                            ++seen[m / 256 * tn + n / 128];
                        }
                        for (int k = 0; k < 4; ++k, v += grid)
                            if (sr::tile_exists(v, tm, tn, split)) return std::printf("behind %d %d %d %d\n", tm, tn, split, v), 1;
                    }
                    for (int c : seen)
                        if (c != 1) return std::printf("%d times: %d x %d, split %d, %d workgroups\n", c, tm, tn, split, grid), 1;
                    ++checked;
                }
    std::printf("%ld\n", checked);
}
"""


def test_every_tile_once(tmp_path):
    (tmp_path / "tiles.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, "-o", str(tmp_path / "tiles"), str(tmp_path / "tiles.cpp")], check=True)
    r = subprocess.run([str(tmp_path / "tiles")], capture_output=True, text=True)
    assert r.returncode == 0 and int(r.stdout) > 10000, r.stdout


def test_rows_per_tile(tmp_path):
    """The rows of an FP6 tile: a multiple of 16 above half of it, no row left out, no empty row of tiles."""
    (tmp_path / "rows.cpp").write_text(r"""
#include "gemm_rules.h"
#include <cstdio>
#include <initializer_list>
int main()
{
    int fewer = 0;
    for (int bm : {128, 192, 256})
        for (long M = 1; M <= 20000; ++M) {
            const long step = sr::f6_row_step(M, bm), tiles = (M + bm - 1) / bm;
            if (step > bm || step * tiles < M || step * (tiles - 1) >= M) return std::printf("%ld rows, %d: %ld\n", M, bm, step), 1;
            if (step < bm && (step % 16 || step <= bm / 2 || (step + 31) / 32 >= bm / 32)) return std::printf("%ld rows, %d: %ld\n", M, bm, step), 1;
            fewer += step < bm;
        }
    std::printf("%d\n", fewer);
}
""")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, "-o", str(tmp_path / "rows"), str(tmp_path / "rows.cpp")], check=True)
    r = subprocess.run([str(tmp_path / "rows")], capture_output=True, text=True)
    assert r.returncode == 0 and int(r.stdout) > 500, r.stdout


def test_paired_tails_follow_the_compute_units(tmp_path):
    """Tiles of 32 x 64, whose paired kernel has room for one workgroup per compute unit, pair while there are no more tiles than those."""
    (tmp_path / "pairs.cpp").write_text(r"""
#include "gemm_rules.h"
#include <cstdio>
int main()
{
    int both = 0;
    for (int cus = 32; cus <= 512; cus *= 2)
        for (int tm = 1; tm <= 20; ++tm)
            for (int tn = 1; tn <= 300; ++tn) {
                const bool pairs = sr::f6_pairs_tails(tm, tn, 2, 4, cus);
                if (pairs != (tm > 2 && tm * tn <= cus)) return std::printf("%d x %d tiles, %d units\n", tm, tn, cus), 1;
                if (sr::f6_pairs_tails(tm, tn, 4, 4, cus) != (tm > 2)) return std::printf("64 x 64, %d x %d tiles\n", tm, tn), 1;
                both += pairs;
            }
    std::printf("%d\n", both);
}
""")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, "-o", str(tmp_path / "pairs"), str(tmp_path / "pairs.cpp")], check=True)
    r = subprocess.run([str(tmp_path / "pairs")], capture_output=True, text=True)
    assert r.returncode == 0 and int(r.stdout) > 100, r.stdout
