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
        const int N = atoi(v[i + 1]), K = atoi(v[i + 2]), mid = svdq::e3m2_mid_shape(M, N, K, true, 256, atoi(v[i + 3]) != 0);
        const int alone = svdq::e3m2_mid_shape(M, N, K, false, 256, atoi(v[i + 3]) != 0);
        int fits = 1;
        if (mid >= 0) {
            const svdq::E3m2Mid& m = svdq::E3M2_MID[mid];
            fits = svdq::e3m2_mid_groups(m, K) >= m.slots && svdq::busiest_xcd((int)((M + m.bm - 1) / m.bm), (N + m.bn - 1) / m.bn) <= 32;
        }
        const int teams = K >= 2048 && svdq::busiest_xcd((int)((M + 127) / 128), N / 128) <= 32;          // of the 128 x 128 kernel
        printf("%ld %d %d %d %d %d\\n", rows, bad + (rows && most > (mt * nt + 7) / 8), mid, alone, fits, teams);
    }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("e3m2_plan")
    (d / "driver.hip").write_text(DRIVER)
    subprocess.run([HIPCC, "--cuda-host-only", "-std=c++17", "-O1", "-I", CSRC, str(d / "driver.hip"), "-o", str(d / "driver")],
                   check=True, capture_output=True, text=True)

    def ask(shapes, whole=False):
        args = [str(v) for s in shapes for v in (*s, 32)[:4]]          # M, N, K and the rank, 32 where a shape names none
        out = subprocess.run([str(d / "driver"), *args], check=True, capture_output=True, text=True).stdout
        return [tuple(map(int, line.split()))[:2 if not whole else None] for line in out.splitlines()]
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


def test_shapes_of_the_gpu_tests(plan):
    """Those of test_walked_tiles (tests/test_gpu_e3m2.py): all tokens on 256 x 256 tiles, one with the last split off, or one tile for
    every CU; of test_walked_layers (tests/test_gpu_layer.py); and of the layers behind a sliced quantise pass, on 128 x 128 tiles."""
    from tests.test_gpu_e3m2 import ONE_EACH, WALKED
    from tests.test_gpu_layer import SLICED
    walked = plan([w[:4] for w in WALKED], whole=True)
    assert [out[0] for out in walked] == [w[0] for w in WALKED[:-1]] + [3072] and all(out[3] == -1 for out in walked)
    assert [out[3] for out in plan([w[:4] for w in ONE_EACH], whole=True)] == [0] * len(ONE_EACH)
    layers = plan([(3300, 5120, 5120, 32), (3300, 5120, 5120, 0), (1216, 13824, 2112, 32), (5376, 3072, 2112, 16)], whole=True)
    assert [out[0] for out in layers] == [3072, 3072, 1024, 5376] and all(out[2] == -1 for out in layers)
    sliced = plan([(M, N, K, r) for M, K, N, r, _, _ in SLICED], whole=True)
    assert all(out[0] == 0 and out[2] == -1 for out in sliced) and [out[5] for out in sliced] == [int(s[5]) for s in SLICED]


# M, N, K, layers with a low-rank term, us on the tiles of the entries of E3M2_MID and on the others
MEASURED_MID = [
    (384, 3072, 5120, (72.1, 46.6, 36.3, 31.8), 38.2), (700, 13824, 3072, (60.7, 68.3, 91.5, 115.5), 66.9), (1024, 5120, 2048, (42.4, 32.6, 42.8, 59.8), 36.3),
    (1024, 5120, 5120, (76.9, 56.4, 68.8, 93.0), 61.3), (1024, 13824, 3072, (99.0, 99.4, 115.5, 151.0), 68.3), (1500, 2048, 1024, (29.1, 22.5, 30.4, 36.4), 20.8),
    (1500, 3072, 5120, (75.9, 50.8, 66.0, 73.3), 59.5), (1500, 5120, 5120, (78.2, 87.3, 92.8, 128.4), 67.2), (2048, 5120, 2048, (44.3, 52.2, 74.1, 94.1), 48.0),
    (2048, 1024, 5120, (74.4, 48.9, 38.5, 51.5), 40.5), (2048, 3072, 5120, (77.4, 56.9, 69.5, 91.4), 63.1), (2048, 5120, 5120, (84.3, 93.4, 120.2, 148.3), 94.2),
    (2048, 13824, 3072, (148.1, 154.0, 190.9, 266.3), 116.2), (3000, 3072, 5120, (86.1, 95.6, 102.7, 135.6), 96.7), (3000, 5120, 5120, (149.1, 139.6, 174.6, 225.4), 107.4),
    (4100, 1024, 5120, (82.0, 57.7, 70.5, 93.7), 64.7), (4100, 13824, 3072, (233.5, 280.4, 369.6, 564.3), 219.1),
]


def test_middling_tokens_near_the_fastest(plan):
    """No choice more than 4 % from the fastest of the five."""
    for (M, N, K, mids, others), out in zip(MEASURED_MID, plan([m[:3] for m in MEASURED_MID], whole=True)):
        took = mids[out[2]] if out[2] >= 0 else others
        assert took <= 1.04 * min(*mids, others), (M, N, K, out[2])


def test_tiles_of_one_team_have_h_summed_ahead(plan):
    """K >= 2048, but more than a tile for every CU: their launch for h's slices counts (packed, M = 833, K = 11328: 154 -> 147 us)."""
    assert [out[2] for out in plan([(785, 12032, 9984, 16), (833, 12288, 11328, 32), (833, 12032, 13568, 16)], whole=True)] == [0, 0, 0]


def test_middling_tiles_are_what_the_kernel_takes(plan):
    """A tile for every CU at most, K loops as long as the rings; without teams only the tile that does not split K.  And the
    shapes of tests/test_gpu_layer.py take the tiles that they are there for."""
    shapes = [(M, N, K, r) for M in (1, 64, 129, 700, 2047, 5000, 75600) for N in (128, 640, 2176, 5120, 13824) for K in (64, 320, 576, 1088, 13824) for r in (0, 32)]
    for s, out in zip(shapes, plan(shapes, whole=True)):
        assert out[4] == 1 and out[3] in (-1, 0), (s, out)
    from tests.test_gpu_layer import MIDDLING
    assert [out[2] for out in plan([(M, N, K, r) for M, K, N, r, _ in MIDDLING], whole=True)] == [m[4] for m in MIDDLING]
