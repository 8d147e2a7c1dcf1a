"""The E3M2 GEMM's split of its tokens between 256 x 256 and 128 x 128 tiles (csrc/svdq_e3m2_plan.h, host code), and the
order in which the walking blocks take their tiles (csrc/svdq_tiles.h)."""
import subprocess

import pytest

from paper_2605_27003_amd.build import CSRC, HIPCC

# M, N, K, us with every token on 256 x 256 tiles, every token on 128 x 128 tiles, split (where it was measured)
MEASURED = [
    (1024, 5120, 512, 16.3, 13.3, None), (2048, 5120, 512, 18.2, 21.2, None), (6400, 5120, 512, 31.8, 43.7, None),
    (16500, 1024, 512, 29.3, 27.0, None), (4700, 13824, 512, 65.7, 78.4, 63.7), (1536, 5120, 1024, 22.0, 16.7, None),
    (4096, 5120, 1024, 41.1, 37.0, 39.7), (9000, 5120, 1024, 64.1, 80.5, None), (2305, 13824, 1024, 60.9, 58.9, 54.9),
    (3300, 5120, 2048, 69.2, 56.0, 54.3), (5000, 4096, 2048, 68.5, 58.6, 60.6), (4700, 13824, 2048, 174.4, 182.8, 159.1),
    (1024, 5120, 5120, 69.2, 41.0, None), (3072, 5120, 5120, 84.6, 91.4, None), (3300, 5120, 5120, 150.1, 117.0, 106.5),
    (4096, 5120, 5120, 149.4, 119.7, None), (6656, 5120, 5120, 231.1, 205.2, 190.4), (16384, 5120, 5120, 425.9, 461.9, None),
    (1213, 13824, 5120, 148.8, 114.5, 103.5), (32768, 1024, 5120, 170.7, 187.0, None), (4700, 13824, 5120, 394.3, 385.6, 352.2),
    (1536, 5120, 13824, 178.3, 114.3, None), (3300, 5120, 13824, 381.0, 286.7, 255.7), (16384, 5120, 13824, 1100.4, 1166.3, None),
    (4700, 13824, 13824, 1019.5, 971.0, 891.7), (16500, 1024, 13824, 381.6, 276.6, 263.2),
]

# the same without a low-rank term
MEASURED_NO_LOWRANK = [
    (8200, 2048, 320, 21.1, 18.7, 21.2), (8200, 2048, 384, 22.7, 19.7, 22.2), (16500, 1024, 384, 22.8, 19.6, 22.2),
    (10239, 1792, 384, 22.7, 20.3, 22.8), (2305, 13824, 512, 37.4, 34.6, 35.2), (3300, 13824, 512, 38.9, 45.5, None),
    (2305, 13824, 640, 42.8, 40.0, 40.5), (4200, 8192, 640, 44.7, 41.7, 43.0), (2305, 5120, 1024, 22.5, 21.7, None),
    (7680, 5120, 1024, 59.8, 61.0, 59.3), (9000, 5120, 1024, 63.7, 72.8, None), (16500, 2048, 1536, 80.2, 70.6, 71.7),
    (6264, 1280, 2048, 34.1, 31.7, None), (1024, 5120, 5120, 70.6, 41.5, None), (3300, 5120, 5120, 144.1, 112.2, 103.4),
    (16384, 5120, 5120, 424.0, 444.2, None), (4700, 13824, 5120, 385.4, 365.2, 341.0), (3072, 5120, 13824, 214.2, 223.8, None),
]

DRIVER = """
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "svdq_e3m2_plan.h"
int main(int n, char** v) {
    for (int i = 1; i + 3 < n; i += 4) {
        const long M = atol(v[i]), rows = svdq::e3m2_walk_rows(M, atoi(v[i + 1]), atoi(v[i + 2]), true, 256, atoi(v[i + 3]) != 0);
        // every tile of those rows once, and the same number (but one) on every XCD
        const int mt = (int)((rows + 255) / 256), nt = atoi(v[i + 1]) / 256;
        const svdq::WalkGrid g = svdq::make_walk_grid(mt, nt);
        std::vector<int> seen(mt * nt);
        int bad = 0, most = 0;
        for (int xcd = 0; xcd < 8 && rows; ++xcd) {
            int own = 0;
            for (int k = 0; k < g.chunk && xcd * g.chunk + k < mt * nt; ++k, ++own) {
                int m, t;
                svdq::walk_tile(g, k * 8 + xcd, m, t);
                if (m < 0 || m >= mt || t < 0 || t >= nt || seen[m * nt + t]++) ++bad;
            }
            most = own > most ? own : most;
        }
        for (int s : seen) bad += s != 1;
        printf("%ld %d\\n", rows, bad + (rows && most > (mt * nt + 7) / 8));
    }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("e3m2_plan")
    (d / "driver.hip").write_text(DRIVER)
    subprocess.run([HIPCC, "--cuda-host-only", "-std=c++17", "-O1", "-I", CSRC, str(d / "driver.hip"), "-o", str(d / "driver")],
                   check=True, capture_output=True, text=True)

    def ask(shapes):
        args = [str(v) for s in shapes for v in (*s, 32)[:4]]          # M, N, K and the rank, 32 where a shape names none
        out = subprocess.run([str(d / "driver"), *args], check=True, capture_output=True, text=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return ask


@pytest.mark.parametrize("measured,r", [(MEASURED, 32), (MEASURED_NO_LOWRANK, 0)])
def test_split_near_the_fastest(plan, measured, r):
    """No choice more than 4 % from the fastest of the three, at every inner dimension, with a low-rank term and without one."""
    for (M, N, K, walk, tiles, split), (rows, bad) in zip(measured, plan([(*m[:3], r) for m in measured])):
        took = walk if rows == M else tiles if rows == 0 else split
        assert took is not None and took <= 1.04 * min(t for t in (walk, tiles, split) if t), (M, N, K, rows)
        assert bad == 0


def test_split_is_what_the_kernels_take(plan):
    """Whole 256-channel tiles and a K loop as long as the ring, whole rows of tiles or all; every tile once."""
    shapes = [(M, N, K) for M in (1, 255, 257, 3300, 32760, 75600) for N in (128, 256, 384, 5120, 13824) for K in (64, 256, 320, 5120)]
    for (M, N, K), (rows, bad) in zip(shapes, plan(shapes)):
        assert bad == 0 and (rows == M or (rows % 256 == 0 and 0 <= rows < M)), (M, N, K, rows)
        if N % 256 or K < 320:
            assert rows == 0


def test_shapes_of_the_gpu_tests_are_walked(plan):
    """The shapes of test_walked_tiles (tests/test_gpu_e3m2.py): all tokens on 256 x 256 tiles, one with the last split off; and
    of test_walked_layers (tests/test_gpu_layer.py)."""
    shapes = [(65537, 256, 320, 32), (65279, 256, 384, 16), (65281, 256, 448, 0), (16001, 1024, 512, 32), (9215, 1792, 576, 0),
              (3072, 5120, 640, 32), (32700, 512, 1024, 16), (3300, 5120, 5120, 32)]
    assert [rows for rows, _ in plan(shapes)] == [s[0] for s in shapes[:-1]] + [3072]
    layers = [(3300, 5120, 5120, 32), (3300, 5120, 5120, 0), (1216, 13824, 2112, 32), (5376, 3072, 2112, 16)]
    assert [rows for rows, _ in plan(layers)] == [3072, 3072, 1024, 5376]
