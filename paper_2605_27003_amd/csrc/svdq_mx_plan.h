// Which tiles an MXFP4 launch takes, and whether its last tokens get a launch of their own (host only).  All tiles give
// the same bits: the order of operations per output is the same.
#pragma once
#include <cstdint>

#include "svdq_kernels.h"
#include "svdq_tiles.h"

namespace svdq {

enum class MxTile { T256x256, T256x128, T128x128 };
struct MxPart {                  // tiles of a launch and its estimated cost, us
    MxTile tile;
    double cost;
};

// The kernel whose blocks walk 256 x 256 tiles needs full 256-channel tiles and a K loop of at least five stages (two more
// than its ring); it then takes every launch of 256 x 256 tiles.
inline bool mx_can_walk(int N, int K) { return N % 256 == 0 && K >= 576; }
// Its tiles are numbered evenly over the XCDs (svdq_tiles.h), so a round is one for each of the `walkers` blocks.  Measured, us:
// 240 tiles 15.7, 17.6, 24.1, 45, 104 at K = 640, 1024, 2048, 5120, 13824, 260 tiles 21.7, 25.3, 36, 70, 165, 1280 tiles 57, 72,
// 110, 217, 530: a round that leaves CUs idle takes less, as the clock rises.
inline double mx_walk_cost(int64_t tiles, int K, int walkers, bool lowrank = true) {
    const double round = (lowrank ? 6.1 : 4.6) + 35.8 * (K / 5120.0), full = (double)(tiles / walkers), f = (double)(tiles % walkers) / walkers;
    return 4.45 + round * (full + (f == 0.0 ? 0.0 : f <= 0.65 ? 0.52 + 0.37 * f : 0.76 + 0.24 * (f - 0.65) / 0.35));
}

// Cheapest tile for `rows` tokens.  A launch of tiles with blocks of their own takes what its busiest XCD takes: whole blocks
// per CU (with several blocks on a CU sharing it), or, where every CU of it is busy throughout and the clock falls, its tiles
// at a lower rate.  A block takes its start and end and then its share of K.  Fitted to 66 shapes at each of K = 384, 512,
// 576, 768, 1024, 1536, 2048, 3328, 5120, 13824, us a block with k = K / 5120, and the rate on a full chip (in brackets:
// without a low-rank term, which is most of what the tiles of four waves begin with):
//   128 x 128   1.87 (0.9) + 10.3 k, 1.09 (1.14)    four waves, three blocks fit a CU
//   256 x 128   4.4 (2.34) + 17.15 k, 1.05 (1.09)   four waves, two blocks; 17 % more for many tokens where XCDs own channels and each reads all of them
//   256 x 256   as above where its blocks can walk; otherwise 9.3 (5.3) + 40 k, 1.15, one block of eight waves
// Choices are within 0.4 % of the fastest tile on average with a low-rank term and 0.7 % without one.  Where estimates are even
// (2 %), tiles are walked: beside a quantise pass those lose less than others.
// Per element the large tiles are a quarter cheaper at K = 5120, but M = 768, N = 5120 is 60 of them on 256 CUs (32 us
// against 18 with 240 tiles of 128 x 128), and with a short K loop and no low-rank term the smaller ones win even on a full
// chip: M = 10240, N = 5120, K = 1024, us on 256 x 256, 256 x 128, 128 x 128: 53.8, 58.2, 57.2, and 49, 43.9, 46.3 without it.
inline MxPart mx_best(int64_t rows, int N, int K, int walkers, bool lowrank = true) {
    const double k = K / 5120.0;
    auto cost = [&](int bm, int bn, double fixed, double ends, double loop, double full, double idle) {
        const int n = busiest_xcd((int)((rows + bm - 1) / bm), N / bn);
        if (5 * n <= 3 * CUS_PER_XCD) return fixed + ends + idle * loop * k;
        const double whole = (n + CUS_PER_XCD - 1) / CUS_PER_XCD, rate = full * n / CUS_PER_XCD;
        return fixed + (ends + loop * k) * (whole > rate ? whole : rate);
    };
    const int m256 = (int)((rows + 255) / 256);
    MxPart best{MxTile::T128x128, cost(128, 128, 3.3, lowrank ? 1.87 : 0.9, 10.3, lowrank ? 1.09 : 1.14, 0.82)};
    const double wide = (rows > 6144 && make_tile_grid(m256, N / 128).nmajor) ? 1.17 : 1.0;
    const double c2 = cost(256, 128, 3.5, wide * (lowrank ? 4.4 : 2.34), wide * 17.15, lowrank ? 1.05 : 1.09, 0.91);
    if (c2 < best.cost) best = MxPart{MxTile::T256x128, c2};
    if (N % 256 == 0) {
        const double c1 = mx_can_walk(N, K) ? mx_walk_cost((int64_t)m256 * (N / 256), K, walkers, lowrank) : cost(256, 256, 1.5, lowrank ? 9.3 : 5.3, 40.0, 1.15, 0.87);
        if (c1 <= 1.02 * best.cost) best = MxPart{MxTile::T256x256, c1};
    }
    return best;
}

// The few-token kernel (svdq_small.hip) on the last `rows` tokens
inline double mx_few_cost(int64_t rows, int N, int K) {
    return 2.0 + (0.010 + 0.028 * (K / 5120.0)) * (double)((rows + 63) / 64) * (double)((N + 63) / 64);
}

// Tokens of the first launch (a multiple of 256, or all of them): leaving the last tokens to a launch of their own on
// smaller tiles pays where they would open another round of blocks for themselves (M = 4700, N = K = 13824: 1026 tiles of
// 256 x 256, 475 us, and 434 with the last 92 or 1116 tokens on smaller ones) and that round is longer than what a launch adds to its
// tiles.  Tried: what fits one or two full rounds less, and the last twelve rows of tiles.  The rest never takes 256 x 256 tiles.
// `tail_cost`: what a launch for the rest costs, in the unit of mx_best.
struct MxSplit {
    int64_t rows;
    double cost;
};
template <class TailCost>
MxSplit mx_split(int64_t M, int N, int K, int walkers, bool lowrank, TailCost tail_cost) {
    const int64_t mtiles = (M + 255) / 256;
    MxSplit best{M, mx_best(M, N, K, walkers, lowrank).cost};
    auto consider = [&](int64_t mt) {
        if (mt < 1 || mt >= mtiles || mx_best(M - mt * 256, N, K, walkers, lowrank).tile == MxTile::T256x256) return;
        const double c = mx_best(mt * 256, N, K, walkers, lowrank).cost + tail_cost(M - mt * 256) + 1.5;
        if (c < best.cost) best = MxSplit{mt * 256, c};
    };
    if (mx_can_walk(N, K)) {
        const int nt = N / 256;
        const int64_t rounds = (mtiles * nt + walkers - 1) / walkers;
        consider((rounds - 1) * walkers / nt);
        consider((rounds - 2) * walkers / nt);
    }
    for (int64_t mt = mtiles - 1; mt >= mtiles - 12; --mt) consider(mt);
    return best;
}

// The rest of a layer's tokens takes the few-token kernel or tiles.
inline double mx_rest_cost(int64_t M, int64_t rest, int N, int K, int walkers, bool lowrank = true) {
    const double few = mx_few_cost(rest, N, K), tiles = mx_best(rest, N, K, walkers, lowrank).cost;
    return small_shape(rest, N, K) && small_reach(M, N, K) && few < tiles ? few : tiles;
}
// Tokens of a layer ahead of that rest
inline int64_t mx_layer_split(int64_t M, int N, int K, int walkers, bool lowrank = true) {
    return mx_split(M, N, K, walkers, lowrank, [&](int64_t rest) { return mx_rest_cost(M, rest, N, K, walkers, lowrank); }).rows;
}
// ... and of its tile launches: all of them, unless the rest is for the few-token kernel
inline int64_t mx_tile_rows(int64_t M, int N, int K, int walkers, bool lowrank = true) {
    const int64_t rows = mx_layer_split(M, N, K, walkers, lowrank);
    return rows < M && mx_rest_cost(M, M - rows, N, K, walkers, lowrank) < mx_best(M - rows, N, K, walkers, lowrank).cost ? rows : M;
}

// Slices of K in the quantise pass of a layer whose GEMM is one of the tile kernels, `row_blocks` <= 128 blocks of 32 tokens.
// A block's eight waves take a pair of groups each at a time; such a step takes 3.5 to 4 us, about 1.3 times that and half a
// step more where CUs have two blocks, and the launch that adds up the slices about 0.8 of a step.  Against powers of two for
// a block per CU at most, as the few-token path takes them (73 row blocks: 2 slices of 20 pairs, 3 steps), whole layers, us:
// K = 5120: M = 1040, N = 5120 40.2 -> 38; 2800 60.9 -> 57.9; 2305, N = 13824 112.4 -> 108.5; K = 13824: M = 2305, N = 1024
// 71.2 -> 58.1, M = 1500, N = 2048 58.0 -> 55.1; K = 1024 (no slices): M = 1300, N = 4096 20.4 -> 19.6.
inline int mx_slices(int row_blocks, int groups) {
    const int pairs = (groups + 1) / 2;
    int best = 1;
    double least = 1e30;
    for (int s = 1; s <= SMALL_SLICES; ++s) {
        if (s > 1 && (s * row_blocks > 512 || groups / s < 8)) break;
        const int steps = ((pairs + s - 1) / s + 7) / 8;
        const double c = (s * row_blocks > 256 ? 1.3 * steps + 0.5 : steps) + (s > 1 ? 0.8 : 0.0);
        if (c <= least) {                                   // as many steps in more slices: more CUs load
            least = c;
            best = s;
        }
    }
    return best;
}

}  // namespace svdq
