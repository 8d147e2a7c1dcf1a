"""Which tokens of an MXFP4 launch the tile-walking kernel takes (csrc/svdq_mx_plan.h, host code), against times measured
with blocks of their own for every tile (or none) and with the walking kernel, its tiles numbered evenly over the XCDs."""
import subprocess

import pytest

from paper_2605_27003_amd.build import CSRC, HIPCC

# M, N, K, us without the walking kernel below 512 tiles, us as it is now
MEASURED = [
    (3072, 5120, 640, 18.7, 16.6), (3300, 5120, 640, 20.2, 20.1), (6400, 5120, 640, 31.2, 25.2), (9000, 5120, 640, 41.4, 32.6),
    (2048, 5120, 1024, 18.5, 15.7), (4096, 5120, 1024, 24.6, 24.8), (2304, 13824, 1024, 35.7, 29.7), (4700, 13824, 1024, 69.1, 61.6),
    (5000, 5120, 2048, 48.4, 39.0), (3300, 5120, 2048, 32.8, 32.7), (6400, 5120, 5120, 109.1, 85.0), (3300, 5120, 5120, 64.3, 58.2),
    (9000, 5120, 5120, 139.1, 118.7), (2305, 13824, 5120, 100.0, 92.2), (4096, 5120, 13824, 160.0, 147.7),
]

DRIVER = """
#include <cstdio>
#include <cstdlib>
#include "svdq_mx_plan.h"
int main(int n, char** v) {
    for (int i = 1; i + 2 < n; i += 3) {
        const long M = atol(v[i]);
        const int N = atoi(v[i + 1]), K = atoi(v[i + 2]);
        const long rows = svdq::mx_layer_walk_rows(M, N, K, 256);
        const double c = rows ? svdq::mx_walk_cost((rows + 255) / 256 * (N / 256), K, 256) +
                                    (rows < M ? 2.0 + svdq::mx_rest_cost(M, M - rows, N, K, 256) : 0.0) : 0.0;
        printf("%ld %.2f\\n", rows, c);
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
        args = [str(v) for s in shapes for v in s]
        out = subprocess.run([str(d / "driver"), *args], check=True, capture_output=True, text=True).stdout
        return [(int(a), float(b)) for a, b in (line.split() for line in out.splitlines())]
    return ask


def test_cost_of_what_is_walked(plan):
    """Where tokens are walked, the estimate is within an eighth of the measured time, and the time no more than before."""
    walked = 0
    for (M, N, K, before, now), (rows, cost) in zip(MEASURED, plan([r[:3] for r in MEASURED])):
        if rows:
            walked += 1
            assert abs(cost - now) <= now / 8, (M, N, K, cost)
        assert now <= 1.02 * before
    assert walked >= 9


def test_walked_tokens_are_what_the_kernel_takes(plan):
    shapes = [(M, N, K) for M in (1, 257, 3300, 32760, 75600) for N in (128, 256, 384, 5120, 13824) for K in (64, 512, 576, 5120)]
    for (M, N, K), (rows, _) in zip(shapes, plan(shapes)):
        assert rows == M or (rows % 256 == 0 and 0 <= rows < M), (M, N, K, rows)
        if N % 256 or K < 576:
            assert rows == 0
