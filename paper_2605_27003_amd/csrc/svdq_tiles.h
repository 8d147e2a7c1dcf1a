// Order in which the GEMM grids take their output tiles.
//
// Consecutive block ids go round-robin to the chip's 8 XCDs, each with an L2 of its own, so a tile order decides
// which tiles share an L2 and how evenly the XCDs are loaded.  Two orders, both a pure function of the block id:
//   token-major   XCD x owns the token tiles x, x + 8, ... and walks them eight at a time across the channel tiles
//                 (the eight blocks an XCD starts together share one weight tile; the activation tiles of its eight
//                 token tiles stay in its L2).  Even when there are many token tiles; with few, the XCDs whose
//                 residue classes are empty or short idle.
//   channel-major XCD x owns the channel tiles x, x + 8, ... and runs all token tiles of one before the next (its
//                 blocks share that weight tile).  For few token tiles and many channel tiles.
// The launcher takes the channel-major order when it lowers the largest share of an XCD by a tenth or more.
#pragma once
#include <hip/hip_runtime.h>

namespace svdq {

struct TileGrid {
    int mtiles, ntiles, nmajor;
    int mt0;                     // first token tile (a launch may cover a part of the tokens)
};

inline TileGrid make_tile_grid(int mtiles, int ntiles, int mt0 = 0) {
    const long long by_m = (long long)((mtiles + 7) / 8) * ntiles;       // blocks of the busiest XCD, token-major
    const long long by_n = (long long)((ntiles + 7) / 8) * mtiles;       // channel-major
    return TileGrid{mtiles, ntiles, by_n * 10 <= by_m * 9 ? 1 : 0, mt0};
}

// tiles of the busiest XCD: what a launch is waited for, in blocks per compute unit (CUS_PER_XCD of them)
constexpr int CUS_PER_XCD = 32;
inline int busiest_xcd(int mtiles, int ntiles) {
    const TileGrid g = make_tile_grid(mtiles, ntiles);
    return g.nmajor ? ((ntiles + 7) / 8) * mtiles : ((mtiles + 7) / 8) * ntiles;
}

// number of block ids (some of them name no tile: tile_of returns false)
__host__ __device__ inline int tile_ids(const TileGrid& g) {
    return g.nmajor ? ((g.ntiles + 7) / 8) * 8 * g.mtiles : ((g.mtiles + 7) / 8) * 8 * g.ntiles;
}

// An XCD's ids number its own tiles without gaps; only an XCD that owns fewer token (or channel) tiles than the others
// has ids left over, at its end.  (With the last group of token tiles numbered as if it were full, 7 of 8 ids named no
// tile at mtiles = 8, and the blocks that did all fell on the same few CUs of the XCD's round-robin: M = 1024,
// K = N = 5120 took 103 us where M = 1536 took 57.)
__device__ __forceinline__ bool tile_of(const TileGrid& g, int id, int& mt, int& nt) {
    const int xcd = id & 7, idx = id >> 3;
    if (g.nmajor) {
        const int q = idx / g.mtiles;
        nt = q * 8 + xcd;
        mt = g.mt0 + idx - q * g.mtiles;
        return nt < g.ntiles;
    }
    const int own = (g.mtiles - xcd + 7) >> 3;                           // token tiles of this XCD
    const int sm = idx / (8 * g.ntiles), rem = idx - sm * (8 * g.ntiles);
    const int width = (own - 8 * sm < 8) ? own - 8 * sm : 8;             // token tiles of this group of eight
    if (width <= 0 || rem >= width * g.ntiles) return false;
    if (width == 8) nt = rem >> 3;                                       // a division is 1 % of a kernel that walks tiles
    else nt = rem / width;
    mt = g.mt0 + (sm * 8 + rem - nt * width) * 8 + xcd;
    return true;
}

// The order of a kernel whose blocks walk their tiles with one block per CU: XCD x takes a run of `chunk` consecutive
// tiles, the same number on every XCD (token tiles owned by residue leave an XCD a token tile ahead of the others: 294 x
// 20 tiles are 23.1 rounds of 32 CUs where the runs are 22.97).  Tiles are numbered in groups of eight token tiles across
// the channel tiles, so the 32 tiles that an XCD's CUs hold at once are 8 x 4.
struct WalkGrid {
    int mtiles, ntiles, chunk;
};
inline WalkGrid make_walk_grid(int mtiles, int ntiles) { return WalkGrid{mtiles, ntiles, (mtiles * ntiles + 7) / 8}; }
// tile of block id `id` (id % 8: its XCD), which exists
__host__ __device__ inline void walk_tile(const WalkGrid& g, int id, int& mt, int& nt) {
    const int n = (id & 7) * g.chunk + (id >> 3), sm = n / (8 * g.ntiles), rem = n - sm * (8 * g.ntiles);
    const int width = g.mtiles - 8 * sm < 8 ? g.mtiles - 8 * sm : 8;
    nt = rem / width;
    mt = 8 * sm + rem - nt * width;
}

}  // namespace svdq
