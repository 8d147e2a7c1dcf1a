"""Which layers are one launch, and how that launch lays out its LDS (csrc/svdq_kernels.h, host code)."""
import subprocess

import pytest

from paper_2605_27003_amd.build import CSRC, HIPCC

DRIVER = """
#include <cstdio>
#include <cstdlib>
#include "svdq_kernels.h"
using namespace svdq;
// every layout that small_fused lets through: the largest, and those whose planes are not aligned for what is read from them
int main(int n, char** v) {
    for (int i = 1; i + 4 < n; i += 5) {
        const long M = atol(v[i]);
        const int K = atoi(v[i + 1]), N = atoi(v[i + 2]), r = atoi(v[i + 3]), mx = atoi(v[i + 4]);
        const int shape = small_shape(M, N, K, mx != 0);
        printf("%d %d %d\\n", shape, shape && small_reach(M, N, K) ? small_fused(M, N, K, r, mx != 0) : 0, small_shape(M, N, K, mx != 0, true));
    }
    unsigned most = 0, askew = 0;
    const long Ms[] = {1, 2, 3, 4, 5, 8, 9, 15, 16, 17, 31, 32, 33, 64, 100, 256, 500, 1000, 2048, 4096, 16384};
    for (long M : Ms)
        for (int N = 128; N <= 16384; N += 128)
            for (int K = 64; K <= 8192; K += 64)
                for (int form = 0; form < 6; ++form) {
                    const int r = 16 * (form % 3), kind = small_fused(M, N, K, r, form >= 3);
                    if (kind == FUSED_NONE) continue;
                    const bool spread = kind == FUSED_SPREAD;
                    for (int ni = 1; ni <= (spread ? 1 : 2); ++ni) {
                        const FusedLds a = fused_lds(ni, K, r != 0, spread, spread ? fused_spread(M) : 5);
                        most = a.end() > most ? a.end() : most;
                        const unsigned h = a.tiles + a.hpart, il = h + a.h, lo = il + a.il, hi = lo + a.lo, scale = hi + a.hi, x = scale + a.scale;
                        askew += a.tiles % 16 || h % 16 || il % 16 || lo % 16 || hi % 8 || scale % 4 || x % 16;
                        if (r) askew += a.hpart != FUSED_HPART * 4 || a.h != FUSED_H * 4;
                    }
                }
    printf("%u %u\\n", most, askew);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "driver.hip").write_text(DRIVER)
    subprocess.run([HIPCC, "--cuda-host-only", "-std=c++17", "-O1", "-I", CSRC, str(d / "driver.hip"), "-o", str(d / "driver")],
                   check=True, capture_output=True, text=True)

    def ask(shapes=()):
        args = [str(int(v)) for s in shapes for v in s]
        out = subprocess.run([str(d / "driver"), *args], check=True, capture_output=True, text=True).stdout
        rows = [tuple(map(int, line.split())) for line in out.splitlines()]
        return rows[:-1], rows[-1]
    return ask


def test_one_launch_fits_the_lds_of_a_cu(plan):
    """Every layer that is one launch: 160 KB at most, and 16-byte accesses at multiples of 16."""
    most, askew = plan()[1]
    assert 160640 <= most <= 160 * 1024 and askew == 0


def test_layers_of_the_gpu_tests_are_one_launch(plan):
    from tests.test_gpu_layer import ONE_LAUNCH, ONE_LAUNCH_MX
    for mx, shapes in ((False, ONE_LAUNCH), (True, ONE_LAUNCH + ONE_LAUNCH_MX)):
        kinds = [row[1] for row in plan([(M, K, N, r, mx) for M, K, N, r, _, _ in shapes])[0]]
        assert all(kinds), list(zip(shapes, kinds))
        if not mx:
            assert kinds == [1] * 9 + [2] * 4


def test_mxfp4_without_a_term_at_k_2048(plan):
    """Two launches there for many tokens (M = 1000, N = 512: 9.7 against 11.4 us)."""
    assert [row[1] for row in plan([(1000, K, 512, 0, True) for K in (1984, 2048)] + [(M, 2048, 1024, 0, True) for M in (400, 500)])[0]] == [2, 0, 2, 0]


def test_shapes_of_the_gpu_tests_on_the_few_token_kernel(plan):
    """tests/test_gpu_layer.py: the tile (1: 32 x 32, 2: 64 x 64 or MXFP4's 32 x 64, 0: none) with canonical weights or nibble codes, with
    E3M2 fields, and of MXFP4; two launches each, so that the kernel runs."""
    from tests.test_gpu_layer import FORMS, SHAPES
    want = {(1030, 1024, 640, 32): (2, 2, 2), (448, 2048, 4096, 32): (2, 0, 0), (449, 2048, 4096, 16): (0, 0, 0), (160, 2112, 6144, 0): (2, 2, 2),
            (161, 2112, 6144, 32): (2, 0, 2), (170, 2112, 6272, 16): (2, 2, 2), (150, 5120, 5120, 32): (2, 2, 2), (130, 2112, 9728, 16): (2, 2, 0),
            (8192, 64, 128, 16): (2, 2, 2), (8193, 64, 128, 16): (0, 0, 2), (10240, 64, 128, 32): (0, 0, 2), (10241, 64, 128, 16): (0, 0, 0),
            (65, 2112, 384, 16): (1, 1, 1), (40, 2112, 640, 16): (1, 1, 1), (150, 5120, 5120, 0): (2, 2, 2), (420, 2112, 4096, 0): (2, 0, 0)}
    assert set(want) <= {s[:4] for s in SHAPES} | set(FORMS)
    int4, mx = (plan([(*s, m) for s in want])[0] for m in (False, True))
    assert [(a[0], a[2], b[0]) for a, b in zip(int4, mx)] == list(want.values())
    assert not any(row[1] for row in int4 + mx)
