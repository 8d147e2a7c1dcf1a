// How the E3M2 GEMM takes its tokens: the first of them on 256 x 256 tiles (svdq_e3m2_walk.hip), the rest on 128 x 128
// tiles (svdq_gemm_e3m2.hip).  Host only.  Both give the same bits, unless the 128 x 128 kernel splits K between two teams.
#pragma once
#include <cstdint>

#include "svdq_tiles.h"

namespace svdq {

// Estimated times, us, k = K / 1024, fitted to K = 512, 1024, 2048, 5120, 13824 and twenty shapes each.
// A walking block takes 4.2 + 15.6 k a tile with every CU busy (K = 5120: 426 us for 1280 tiles).  A round that leaves CUs
// idle takes less, as the clock rises: 0.78 of it at a third, 0.82 at five eighths of the CUs.
inline double e3m2_walk_cost(int64_t tiles, int K, int walkers) {
    const double round = 4.2 + 15.6 * (K / 1024.0), full = (double)(tiles / walkers), f = (double)(tiles % walkers) / walkers;
    return 6.0 + round * (full + (f == 0.0 ? 0.0 : f <= 0.65 ? 0.78 + 0.06 * f : 0.82 + 0.18 * (f - 0.65) / 0.35));
}
// 128 x 128 tiles, two blocks per CU: 5 + 8.2 k for a pair, 3 + 4.3 k for a block alone on its CU, or 6 + 3.7 k as two
// teams of waves; K = 5120: 41, 47, 72, 91, 120, 462 us for 1.25, 1.9, 2.5, 3.75, 5, 20 tiles per CU.
inline double e3m2_tiles_cost(int64_t rows, int N, int K, bool teams) {
    const double k = K / 1024.0, pair = 5.0 + 8.2 * k;
    const double n = busiest_xcd((int)((rows + 127) / 128), N / 128) / (double)CUS_PER_XCD;
    const int pairs = (int)(n / 2);
    const double rest = n - 2 * pairs, solo = pairs == 0 && teams && K >= 2048 ? 6.0 + 3.7 * k : 3.0 + 4.3 * k;
    return 4.0 + pairs * pair + (rest > 1 ? pair * (0.78 + 0.22 * (rest - 1)) : rest > 0 ? solo * (0.8 + 0.2 * rest) : 0.0);
}

// Tokens for the 256 x 256 tiles: none, all, or as many whole rows of tiles as fit a number of full rounds of the CUs.  In
// full rounds they take 6 to 27 % less than 128 x 128 tiles (half the bytes from L2 to LDS per output, starts and ends of
// tiles mostly hidden; M = 32760, K = N = 5120: 871 against 945 us), but a round begun for a few tiles costs nearly a whole
// one (M = 3300: 150 against 117 us, and 85 + 27 as 3072 tokens and the rest).
inline int64_t e3m2_walk_rows(int64_t M, int N, int K, bool teams, int walkers) {
    if (N % 256 || K < 320) return 0;                            // whole tiles; a K loop as long as the ring
    const int nt = N / 256;
    const int64_t mt = (M + 255) / 256, rounds = (mt * nt + walkers - 1) / walkers;
    int64_t best = 0;
    double least = e3m2_tiles_cost(M, N, K, teams);
    for (int64_t r = rounds > 3 ? rounds - 2 : 1; r <= rounds; ++r) {
        const int64_t m = r == rounds ? mt : r * walkers / nt;
        if (m == 0) continue;
        const int64_t rows = m >= mt ? M : m * 256;
        const double c = e3m2_walk_cost(m * nt, K, walkers) + (rows < M ? 4.0 + e3m2_tiles_cost(M - rows, N, K, teams) : 0.0);
        if (c < least) {
            least = c;
            best = rows;
        }
    }
    return best;
}

}  // namespace svdq
