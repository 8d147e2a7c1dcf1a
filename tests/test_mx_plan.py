"""The MXFP4 GEMM's choice of tiles and of a launch for the last tokens (csrc/svdq_mx_plan.h, host code): at every
inner dimension, against times measured with each tile forced and no launch split off."""
import os
import subprocess

import pytest

from paper_2605_27003_amd.build import CSRC, HIPCC

# K, M, N, us on 256 x 256, 256 x 128, 128 x 128 tiles
MEASURED = [
    (512, 2048, 5120, 15.6, 15.0, 12.7), (512, 4096, 5120, 28.3, 23.3, 19.7), (512, 9000, 5120, 53.8, 46.5, 37.8),
    (512, 8300, 4096, 42.9, 35.0, 28.6), (512, 2305, 13824, 40.1, 33.5, 28.1), (512, 17000, 1024, 28.0, 23.1, 18.5),
    (512, 16500, 2048, 38.8, 33.5, 28.0), (512, 6200, 10240, 62.3, 56.5, 49.9), (512, 3100, 8192, 28.0, 25.9, 23.2),
    (512, 4200, 3072, 24.9, 15.3, 16.0), (1024, 9000, 5120, 48.8, 60.3, 50.4), (1024, 4200, 3072, 29.2, 18.4, 19.5),
    (1024, 16384, 5120, 72.4, 81.0, 83.8), (1024, 17000, 1024, 32.1, 26.7, 22.8), (2048, 9000, 5120, 74.2, 85.3, 75.2),
    (2048, 768, 5120, 20.2, 13.6, 10.3), (2048, 16384, 5120, 107.7, 118.7, 125.7), (2048, 6200, 10240, 89.1, 105.6, 112.7),
    (5120, 768, 5120, 33.7, 22.5, 17.6), (5120, 4096, 5120, 76.1, 65.1, 65.1), (5120, 9000, 5120, 148.4, 164.9, 147.2),
    (5120, 16384, 5120, 210.1, 229.8, 255.6), (5120, 4200, 3072, 68.4, 48.0, 54.0), (13824, 768, 5120, 70.6, 46.2, 38.5),
    (13824, 16384, 5120, 506.8, 541.8, 603.5), (13824, 4200, 3072, 154.5, 113.6, 129.7), (13824, 1100, 5120, 70.9, 52.2, 54.8),
]

DRIVER = """
#include <cstdio>
#include <cstdlib>
#include "svdq_mx_plan.h"
int main(int n, char** v) {
    for (int i = 1; i + 2 < n; i += 3) {
        const long M = atol(v[i + 1]);
        const int K = atoi(v[i]), N = atoi(v[i + 2]);
        const long rows = svdq::mx_layer_split(M, N, K, 256);
        printf("%d %ld\\n", (int)svdq::mx_best(M, N, K, 256).tile, rows);
    }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("mx_plan")
    (d / "driver.hip").write_text(DRIVER)
    subprocess.run([HIPCC, "--cuda-host-only", "-std=c++17", "-O1", "-I", CSRC, str(d / "driver.hip"), "-o", str(d / "driver")],
                   check=True, capture_output=True, text=True)

    def ask(shapes):
        args = [str(v) for s in shapes for v in s]
        out = subprocess.run([str(d / "driver"), *args], check=True, capture_output=True, text=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return ask


def test_tile_near_the_fastest_at_every_inner_dimension(plan):
    """No choice more than 10 % from the fastest tile (the costs of K = 5120 at every K: up to 25 %)."""
    for row, (tile, _) in zip(MEASURED, plan([r[:3] for r in MEASURED])):
        times = row[3:]
        assert times[tile] <= 1.10 * min(times), (row, tile)


def test_launch_split_off_where_it_pays(plan):
    """A round of blocks saved is worth its share of K; a launch costs the same at any K.  Measured, whole against split,
    us: M = 2305, N = 13824, K = 1024: 40 / 46, K = 5120: 107 / 99; M = 9000, N = 5120, K = 2048: 74 / 81, K = 5120: 148 / 139."""
    shapes = [(1024, 2305, 13824), (5120, 2305, 13824), (2048, 9000, 5120), (5120, 9000, 5120), (512, 9000, 5120)]
    rows = [r for _, r in plan(shapes)]
    assert rows == [2305, 2304, 9000, 6144, 9000]
    for K, M, N in shapes:
        for m in (1, 255, 256, 257, M):
            (tile, r), = plan([(K, m, N)])
            assert r == m or (0 < r < m and r % 256 == 0)


SLICES_DRIVER = """
#include <cstdio>
#include "svdq_mx_plan.h"
int main() {
    for (int rb = 1; rb <= 128; ++rb)
        for (int groups = 1; groups <= 256; ++groups) printf("%d ", svdq::mx_slices(rb, groups));
}
"""


def test_slices_of_the_quantise_pass(tmp_path):
    """Never more slices than partial sums are summed, a group per wave and slice, two blocks of 32 tokens per CU at most; and
    the ones measured to be the fastest (K = 5120 and 13824)."""
    (tmp_path / "driver.hip").write_text(SLICES_DRIVER)
    subprocess.run([HIPCC, "--cuda-host-only", "-std=c++17", "-O1", "-I", CSRC, str(tmp_path / "driver.hip"), "-o", str(tmp_path / "driver")],
                   check=True, capture_output=True, text=True)
    flat = [int(v) for v in subprocess.run([str(tmp_path / "driver")], check=True, capture_output=True, text=True).stdout.split()]
    got = {(1 + i // 256, 1 + i % 256): s for i, s in enumerate(flat)}
    for (rb, groups), s in got.items():
        assert s == 1 or (1 < s <= 8 and s * rb <= 512 and groups // s >= 8), (rb, groups, s)
    # 1040, 1536, 2305, 2800 tokens; K = 13824; K = 1024
    assert [got[rb, 80] for rb in (33, 48, 73, 88)] == [7, 5, 7, 5]
    assert got[73, 216] == 7 and got[41, 16] == 1
