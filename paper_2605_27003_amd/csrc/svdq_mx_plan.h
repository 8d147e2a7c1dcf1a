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

// The tile-walking kernel needs full 256-channel tiles and a K loop of at least five stages (two more than its ring); with
// two tiles and more for each of its `walkers` blocks its tiles cost less than blocks of their own.
inline bool mx_walks(int mtiles, int N, int K, int walkers) {
    return N % 256 == 0 && K >= 576 && (int64_t)mtiles * (N / 256) >= 2 * (int64_t)walkers;
}

// Cheapest tile for `rows` tokens.  A launch takes what its busiest XCD takes: whole blocks per CU (with several blocks on a
// CU sharing it), or, where every CU of it is busy throughout and the clock falls, its tiles at a lower rate; with 40 % of
// the CUs idle the clock rises.  A block takes its start and end and then its share of K.  Measured for K = 512, 1024, 2048,
// 5120, 13824 and eighteen shapes, us a block with k = K / 5120 (and the factors on a full chip, and of k on an idle one):
//   128 x 128   1.8 + 11.5 k (1.07, 1)     four waves, three blocks fit a CU
//   256 x 128   4.4 + 17.3 k (1.03, 0.87)  four waves, two blocks; 15 % more for many tokens where XCDs own channels and each reads all of them
//   256 x 256   10 + 28 k (1.15, 0.87)     eight waves, one block; 6 + 31 k as one block per CU that walks its tiles (9 + 29 k where XCDs own channels)
// Per element the large tiles are a quarter cheaper at K = 5120, but M = 768, N = 5120 is 60 of them on 256 CUs (34 us
// against 18 with 240 tiles of 128 x 128), and with a short K loop their starts and ends cost more than that: M = 9000,
// N = 5120 takes 54 us on 256 x 256, 47 on 256 x 128 and 38 on 128 x 128 at K = 512, and 148, 165 and 147 at K = 5120.
inline MxPart mx_best(int64_t rows, int N, int K, int walkers) {
    const double k = K / 5120.0;
    auto cost = [&](int bm, int bn, double fixed, double ends, double loop, double full, double idle) {
        const int n = busiest_xcd((int)((rows + bm - 1) / bm), N / bn);
        if (5 * n <= 3 * CUS_PER_XCD) return fixed + ends + idle * loop * k;
        const double whole = (n + CUS_PER_XCD - 1) / CUS_PER_XCD, rate = full * n / CUS_PER_XCD;
        return fixed + (ends + loop * k) * (whole > rate ? whole : rate);
    };
    const int m256 = (int)((rows + 255) / 256);
    MxPart best{MxTile::T128x128, cost(128, 128, 5.0, 1.8, 11.5, 1.07, 1.0)};
    const double wide = (rows > 6144 && make_tile_grid(m256, N / 128).nmajor) ? 1.15 : 1.0;
    const double c2 = cost(256, 128, 4.0, wide * 4.4, wide * 17.3, 1.03, 0.87);
    if (c2 < best.cost) best = MxPart{MxTile::T256x128, c2};
    if (N % 256 == 0) {
        const bool walks = mx_walks(m256, N, K, walkers), nmajor = make_tile_grid(m256, N / 256).nmajor;
        const double c1 = !walks ? cost(256, 256, 1.5, 10.0, 28.0, 1.15, 0.87) : nmajor ? cost(256, 256, 1.5, 9.0, 29.0, 1.15, 0.87)
                                                                                        : cost(256, 256, 1.5, 6.0, 31.0, 1.15, 0.87);
        if (c1 <= best.cost) best = MxPart{MxTile::T256x256, c1};
    }
    return best;
}

// The few-token kernel (svdq_small.hip) on `rows` tokens
inline double mx_few_cost(int64_t rows, int N, int K) {
    return 5.0 + (0.010 + 0.028 * (K / 5120.0)) * (double)((rows + 63) / 64) * (double)((N + 63) / 64);
}

// Tokens of the first launch (a multiple of 256, or all of them): leaving the last tokens to a launch of their own on
// smaller tiles pays where they would open another round of blocks for themselves (M = 2305, N = 13824: 70 tiles of
// 256 x 256 on the busiest XCD's 32 CUs, 63 without the one row beyond 2304) and that round is longer than a launch, which
// takes about 2 us at any K.  `tail_cost`: what a launch for the rest costs, in the unit of mx_best.
struct MxSplit {
    int64_t rows;
    double cost;
};
template <class TailCost>
MxSplit mx_split(int64_t M, int N, int K, int walkers, TailCost tail_cost) {
    const int mtiles = (int)((M + 255) / 256);
    MxSplit best{M, mx_best(M, N, K, walkers).cost};
    for (int mt = mtiles - 1; mt >= 1 && mt >= mtiles - 12; --mt) {
        const double c = mx_best((int64_t)mt * 256, N, K, walkers).cost + tail_cost(M - (int64_t)mt * 256) + 2.0;
        if (c < 0.985 * best.cost) best = MxSplit{(int64_t)mt * 256, c};
    }
    return best;
}

// The kernel whose blocks walk 256 x 256 tiles takes the tokens, or as many rows of tiles as fit full rounds of the CUs, where that is the cheapest.  Its tiles are
// numbered evenly over the XCDs (svdq_tiles.h), so a round is 256 of them: 4.3 + 38 k us, k = K / 5120, and less for a
// round that leaves CUs idle, whose clock rises (0.6 of it with a few tiles, 0.71 at five eighths of the CUs).  Measured, us:
// 256 tiles 16.5, 19.2, 26.5, 50.7, 115 at K = 640, 1024, 2048, 5120, 13824, 260 tiles 23, 26, 38, 74, 178, 1280 tiles 53, 68,
// 106, 220, 539.  With fewer than two fifths of the CUs in the last round the smaller tiles have to look a tenth slower: their
// cost is a tenth too high there at K <= 2048 (M = 3300, N = 5120: 22 us at K = 1024, 33 at K = 2048).
inline double mx_walk_cost(int64_t tiles, int K, int walkers) {
    const double round = 4.3 + 37.8 * (K / 5120.0), full = (double)(tiles / walkers), f = (double)(tiles % walkers) / walkers;
    return 7.5 + round * (full + (f == 0.0 ? 0.0 : f <= 0.65 ? 0.6 + 0.18 * f : 0.715 + 0.285 * (f - 0.65) / 0.35));
}
template <class TailCost>
int64_t mx_walk_rows(int64_t M, int N, int K, int walkers, TailCost tail_cost) {
    if (N % 256 || K < 576) return 0;
    const int nt = N / 256;
    const int64_t mt = (M + 255) / 256, rounds = (mt * nt + walkers - 1) / walkers;
    int64_t best = 0;
    double least = mx_split(M, N, K, walkers, tail_cost).cost;
    for (int64_t r = rounds > 3 ? rounds - 2 : 1; r <= rounds; ++r) {
        const int64_t m = r == rounds ? mt : r * walkers / nt;
        if (m == 0) continue;
        const int64_t rows = m >= mt ? M : m * 256;
        const double c = mx_walk_cost(m * nt, K, walkers) + (rows < M ? 2.0 + tail_cost(M - rows) : 0.0);
        const bool few = m * nt % walkers > 0 && 5 * (m * nt % walkers) < 2 * walkers;
        if (c < (few ? 0.9 : 1.0) * least) {
            least = c;
            best = rows;
        }
    }
    return best;
}

// The rest of a layer's tokens takes the few-token kernel or tiles.
inline double mx_rest_cost(int64_t M, int64_t rest, int N, int K, int walkers) {
    const double few = mx_few_cost(rest, N, K), tiles = mx_best(rest, N, K, walkers).cost;
    return small_shape(rest, N, K) && small_reach(M, N, K) && few < tiles ? few : tiles;
}
// Tokens of a layer that are best left to the tile kernels other than the walking one; the rest as above.
inline int64_t mx_layer_split(int64_t M, int N, int K, int walkers) {
    return mx_split(M, N, K, walkers, [&](int64_t rest) { return mx_rest_cost(M, rest, N, K, walkers); }).rows;
}
// ... and the walking one's
inline int64_t mx_layer_walk_rows(int64_t M, int N, int K, int walkers) {
    return mx_walk_rows(M, N, K, walkers, [&](int64_t rest) { return mx_rest_cost(M, rest, N, K, walkers); });
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
