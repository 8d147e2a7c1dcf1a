// How the E3M2 GEMM takes its tokens: the first of them on 256 x 256 tiles (svdq_e3m2_walk.hip), the rest on 128 x 128
// tiles (svdq_gemm_e3m2.hip); or, where they are one tile for every CU at most, on the tiles of svdq_e3m2_mid.hip.  Host only.
// All give the same bits, unless a kernel splits K between teams.
#pragma once
#include <cstdint>

#include "svdq_tiles.h"

namespace svdq {

// Estimated times, us, k = K / 1024, fitted to 41 shapes at each of K = 320, 384, 512, 640, 1024, 2048, 5120, 13824, GEMMs
// and whole layers, with a low-rank term and without one.  The term is most of what a tile begins with: 128 x 128 tiles lose
// 2 us a pair without it, 256 x 256 tiles 1 us (M = 8200, N = 2048, K = 384, walked and 128 x 128: 25.9 and 23.8 with it,
// 23.3 and 19.2 without).
// A walking block takes 4.8 + 15.4 k a tile with every CU busy (K = 5120: 426 us for 1280 tiles).  A round that leaves a
// third of the CUs idle takes 0.83 of it, as the clock rises; one begun for a few tiles costs a whole one.
inline double e3m2_walk_cost(int64_t tiles, int K, int walkers, bool lowrank) {
    const double round = (lowrank ? 4.8 : 3.9) + 15.4 * (K / 1024.0), full = (double)(tiles / walkers), f = (double)(tiles % walkers) / walkers;
    return 4.4 + round * (full + (f == 0.0 ? 0.0 : f <= 0.65 ? 1.0 - 0.27 * f : 0.88 + 0.12 * (f - 0.65) / 0.35));
}
// 128 x 128 tiles, two blocks per CU: 5.3 + 8.3 k for a pair, 3.8 + 3.6 k for a block alone on its CU, or 7.2 + 2.1 k as two
// teams of waves.  Tiles per CU: between those of the busiest XCD and the average (the last blocks of one start early).
inline double e3m2_tiles_cost(int64_t rows, int N, int K, bool teams, bool lowrank) {
    const double k = K / 1024.0, pair = (lowrank ? 5.3 : 3.3) + 8.3 * k;
    const int mtiles = (int)((rows + 127) / 128), ntiles = N / 128;
    const double n = 0.5 * (busiest_xcd(mtiles, ntiles) + (double)mtiles * ntiles / 8) / CUS_PER_XCD;
    const int pairs = (int)(n / 2);
    const double rest = n - 2 * pairs, solo = pairs == 0 && teams && K >= 2048 ? (lowrank ? 7.2 : 4.0) + 2.1 * k : (lowrank ? 3.8 : 2.2) + 3.6 * k;
    return 3.8 + pairs * pair + (rest > 1 ? pair * (0.82 + 0.18 * (rest - 1)) : rest > 0 ? solo * (pairs == 0 ? 1.0 : 0.86 + 0.14 * rest) : 0.0);
}

// Tokens for the 256 x 256 tiles: none, all, or as many whole rows of tiles as fit a number of full rounds of the CUs.  In
// full rounds they take 6 to 27 % less than 128 x 128 tiles (half the bytes from L2 to LDS per output, starts and ends of
// tiles mostly hidden; M = 32760, K = N = 5120: 871 against 945 us), but a round begun for a few tiles costs nearly a whole
// one (M = 3300: 150 against 117 us, and 85 + 27 as 3072 tokens and the rest).
inline int64_t e3m2_walk_rows(int64_t M, int N, int K, bool teams, int walkers, bool lowrank = true) {
    if (N % 256 || K < 320) return 0;                            // whole tiles; a K loop as long as the ring
    const int nt = N / 256;
    const int64_t mt = (M + 255) / 256, rounds = (mt * nt + walkers - 1) / walkers;
    int64_t best = 0;
    double least = e3m2_tiles_cost(M, N, K, teams, lowrank);
    for (int64_t r = rounds > 3 ? rounds - 2 : 1; r <= rounds; ++r) {
        const int64_t m = r == rounds ? mt : r * walkers / nt;
        if (m == 0) continue;
        const int64_t rows = m >= mt ? M : m * 256;
        const double c = e3m2_walk_cost(m * nt, K, walkers, lowrank) + (rows < M ? 2.5 + e3m2_tiles_cost(M - rows, N, K, teams, lowrank) : 0.0);
        if (c < least) {
            least = c;
            best = rows;
        }
    }
    return best;
}

// The kernel for middling numbers of tokens (svdq_e3m2_mid.hip): tokens and channels of a block's tile, teams that split K,
// slots of a team's ring.  Its K loop is as long as the ring at least.
struct E3m2Mid {
    int bm, bn, teams, slots;
    double begin, group, loaded;                                 // us: a tile's start and end, a team's group on an idle chip, more on a full one
};
constexpr E3m2Mid E3M2_MID[] = {{256, 192, 1, 5, 9.1, 0.601, 0.242}, {128, 192, 2, 4, 8.2, 0.612, 0.314}, {128, 96, 4, 3, 8.5, 0.676, 0.390}, {64, 96, 8, 2, 8.0, 0.970, 0.385}};
inline int e3m2_mid_groups(const E3m2Mid& m, int K) { return (K / 64 + m.teams - 1) / m.teams; }
// Which of them a launch of all tokens takes, or -1: the others.  split: K may be split between teams (a whole layer).
// Costs fitted to 95 shapes of M = 96 .. 4100, K = 1024 .. 13824 with a term (2 to 4 %); without one a tile's start is 2 us shorter.
// Only where the tiles are one for every CU at most: further rounds take long.  The others are estimated as above, except that two teams of
// 128 x 128 tiles on a chip that they fill take 9.3 + 3.1 k, and ahead of the others, which do not add up h's slices themselves, that
// takes a launch (1.5 us) for up to 4096 tokens.  Layers, us:
// M = 2048, K = N = 5120 94.2 -> 84.3, M = 1500, N = 3072 59.5 -> 50.8, M = 1024, K = 2048, N = 5120 36.3 -> 32.6;
// 270 random layers that take one 0.94 on average, 0.97 for K < 1024, where nothing was fitted; 12 of them lost more than 2 %, 1.07 at most and
// 1.11 (M = 396, K = 896, N = 2816, 18.3 -> 20.3) below K = 1024.  With less than 1.5 % to gain the others are taken: M = 1500, K = 1024, N = 2048 20.8
// against 22.5, and M = 512, K = N = 5120, whose GEMM alone takes 24.6 us here and 28.8 there but whose layer 37.9 and 38.9.
inline int e3m2_mid_shape(int64_t M, int N, int K, bool split, int walkers, bool lowrank) {
    if (walkers != 8 * CUS_PER_XCD) return -1;
    const int64_t rows = e3m2_walk_rows(M, N, K, split, walkers, lowrank);
    const bool two_teams = split && rows == 0 && K >= 2048 && busiest_xcd((int)((M + 127) / 128), N / 128) <= CUS_PER_XCD;
    double least = 0.0;
    if (rows) {
        least = e3m2_walk_cost((rows + 255) / 256 * (N / 256), K, walkers, lowrank) + (rows < M ? 2.5 + e3m2_tiles_cost(M - rows, N, K, split, lowrank) : 0.0);
    } else if (two_teams) {
        least = (lowrank ? 9.3 : 7.3) + 3.1 * (K / 1024.0);
    } else {
        least = e3m2_tiles_cost(M, N, K, split, lowrank);
    }
    if (!two_teams && split && lowrank && M <= 4096 && K >= 1024) least += 1.5;
    least *= 0.985;
    int best = -1;
    for (int i = 0; i < 4; ++i) {
        const E3m2Mid& m = E3M2_MID[i];
        const int64_t mtiles = (M + m.bm - 1) / m.bm;
        const int ntiles = (N + m.bn - 1) / m.bn;
        if ((m.teams > 1 && !split) || mtiles > 256 || busiest_xcd((int)mtiles, ntiles) > CUS_PER_XCD || e3m2_mid_groups(m, K) < m.slots) continue;
        const double load = (double)mtiles * ntiles / walkers;
        const double c = m.begin - (lowrank ? 0.0 : 2.0) + e3m2_mid_groups(m, K) * (m.group + (load > 0.4 ? m.loaded * (load - 0.4) : 0.0));
        if (c < least) {
            least = c;
            best = i;
        }
    }
    return best;
}

}  // namespace svdq
