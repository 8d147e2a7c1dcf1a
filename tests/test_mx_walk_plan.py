"""How an MXFP4 GEMM divides its tokens between launches, and which of them the tile-walking kernel takes
(csrc/svdq_mx_plan.h, host code), against measured times."""
import subprocess

import pytest

from paper_2605_27003_amd.build import CSRC, HIPCC

# M, N, K, us with all tokens walked, all on the better of the smaller tiles, and divided (None: nothing to divide)
MEASURED = [
    (3072, 5120, 640, 15.6, 17.3, None), (3300, 5120, 640, 21.8, 19.5, 22.3), (6400, 5120, 640, 26.7, 31.7, 35.8),
    (9000, 5120, 640, 35.2, 42.0, 44.9), (2048, 5120, 1024, 16.0, 17.4, None), (4096, 5120, 1024, 26.2, 26.3, 31.6),
    (2304, 13824, 1024, 33.5, 37.0, 42.6), (4700, 13824, 1024, 66.5, 71.7, 65.6), (5000, 5120, 2048, 41.0, 44.7, 48.2),
    (3300, 5120, 2048, 36.1, 33.7, 33.4), (6400, 5120, 5120, 85.8, 106.8, 109.5), (3300, 5120, 5120, 69.6, 64.3, 58.4),
    (9000, 5120, 5120, 124.5, 148.3, 137.7), (10240, 5120, 5120, 151.8, 152.7, 144.5), (2305, 13824, 5120, 110.6, 107.4, 99.3),
    (10239, 1792, 5184, 72.0, 64.1, 62.6), (4096, 5120, 13824, 168.0, 152.5, 155.5), (10240, 5120, 13824, 372.8, 363.5, 345.2),
    (4700, 13824, 13824, 476.8, 472.9, 437.8), (75600, 5120, 13824, 2438.8, 2594.8, 2421.4),
]

DRIVER = """
#include <cstdio>
#include <cstdlib>
#include "svdq_mx_plan.h"
using namespace svdq;
int main(int n, char** v) {
    for (int i = 1; i + 3 < n; i += 4) {
        const long M = atol(v[i]);
        const int N = atoi(v[i + 1]), K = atoi(v[i + 2]);
        const bool lowrank = atoi(v[i + 3]) != 0;
        const MxSplit s = mx_split(M, N, K, 256, lowrank, [&](int64_t rest) { return mx_best(rest, N, K, 256, lowrank).cost; });
        const bool walked = mx_best(s.rows, N, K, 256, lowrank).tile == MxTile::T256x256 && mx_can_walk(N, K);
        printf("%ld %ld %d %.2f %.2f\\n", (long)s.rows, (long)mx_tile_rows(M, N, K, 256, lowrank), (int)walked, s.cost,
               mx_walk_cost((M + 255) / 256 * (N / 256), K, 256, lowrank));
    }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("mx_walk_plan")
    (d / "driver.hip").write_text(DRIVER)
    subprocess.run([HIPCC, "--cuda-host-only", "-std=c++17", "-O1", "-I", CSRC, str(d / "driver.hip"), "-o", str(d / "driver")],
                   check=True, capture_output=True, text=True)

    def ask(shapes):
        """(tokens of the first launch, tokens of a layer's tile launches, whether the first launch walks, its estimate, that of walking all)"""
        args = [str(v) for s in shapes for v in (*s, 32)[:4]]          # M, N, K and the rank, 32 where a shape names none
        out = subprocess.run([str(d / "driver"), *args], check=True, capture_output=True, text=True).stdout
        return [(int(a), int(b), int(c), float(e), float(w)) for a, b, c, e, w in (line.split() for line in out.splitlines())]
    return ask


def test_division_near_the_fastest(plan):
    """What the plan takes is within 4 % of the fastest of the three, and its estimate of the walking kernel, by which it
    judges every launch of that kernel, within an eighth of the measured time."""
    walked = 0
    for (M, N, K, walk, tiles, split), (rows, _, walks, cost, walk_cost) in zip(MEASURED, plan([m[:3] for m in MEASURED])):
        took = split if rows < M else walk if walks else tiles
        assert took is not None and took <= 1.04 * min(t for t in (walk, tiles, split) if t), (M, N, K, rows, walks)
        assert abs(walk_cost - walk) <= walk / 8, (M, N, K, walk_cost)
        if rows == M and walks:
            assert cost == walk_cost
        walked += walks
    assert walked >= 15


def test_shapes_of_the_gpu_tests_are_walked(plan):
    """The shapes of tests/test_gpu_mxfp4.py and tests/test_gpu_fused_next.py that are there for the walking kernel, and of
    tests/test_gpu_layer.py for the few-token kernel behind it."""
    whole = [(1999, 16384, 640, 32), (2590, 5120, 576, 16), (6300, 5120, 576, 0), (2305, 5120, 1088, 32), (5000, 5120, 1088, 16),
             (1100, 32768, 704, 32)]
    assert [(rows, walks) for rows, _, walks, _, _ in plan(whole)] == [(s[0], 1) for s in whole]
    (rows, _, walks, _, _), = plan([(1803, 10240, 1600, 32)])
    assert walks and rows == 1536
    # tests/test_gpu_layer.py: the last token is for the few-token kernel, behind 128 x 128 tiles and behind walked ones
    few = [(2049, 1408, 1088, 32), (6401, 2560, 576, 16)]
    assert [tiles for _, tiles, *_ in plan(few)] == [2048, 6400]
    assert [walks for _, _, walks, *_ in plan([(m // 256 * 256, n, k, r) for m, n, k, r in few])] == [0, 1]


def test_divisions_are_what_the_kernels_take(plan):
    """Whole rows of 256 tokens, or all of them; what is left to the few-token kernel are a layer's last tokens."""
    shapes = [(M, N, K, r) for M in (1, 255, 257, 3300, 32760, 75600) for N in (128, 256, 384, 5120, 13824) for K in (64, 512, 576, 5120) for r in (0, 32)]
    for (M, N, K, _), (rows, tiles, walks, _, _) in zip(shapes, plan(shapes)):
        assert rows == M or (rows % 256 == 0 and 0 < rows < M), (M, N, K, rows)
        assert tiles == M or (tiles % 256 == 0 and 0 < tiles < M), (M, N, K, tiles)
        assert not walks or (N % 256 == 0 and K >= 576)
