// asd_mm_tiles.h -- tile widths of the one-launch micromagnetic step and the
// rule that takes one of them or the stage kernels (host and device).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

namespace asd {

constexpr int kMMThreads = 1024, kMMCells = 2, kMMHalo = 3;
// Tile widths.  Their widened columns fit kMMThreads * kMMCells cells up to 16,
// 14, 10, 8, 4 and 2 planes, and the boxes of FP32 the LDS as far; those of FP64
// (twice the bytes) up to 14, 11, 8, 6 and 2 planes, and the widest none.
constexpr int kMMTiles[] = {5, 6, 8, 10, 16, 26};
constexpr int kMMTileMax64 = 16;  // the widest in FP64
constexpr size_t kMMTileLds = 128 * 1024;

inline size_t mm_tile_lds(int tile, int nz, int elem)
{
    const size_t B = tile + 2 * kMMHalo + 2;
    return 2 * 3 * B * B * ((size_t)nz + 2) * elem;
}

// Modelled time (us) of a step in tiles of width t, n tiles: rounds of as many
// workgroups as a CU holds (two by threads, less by LDS), each a fixed latency
// and its cells; fitted to 129 meshes of 600 cells to 14.4M on MI355X, 6 % rms.
inline double mm_tile_us(int t, int64_t n, int nz, int elem)
{
    const double nw = (double)(t + 2 * kMMHalo) * (t + 2 * kMMHalo) * nz;
    const double one = elem == 8 ? 3.7 + 7.2e-3 * nw : 3.0 + 4.9e-3 * nw;
    const int per_cu = (int)std::min<size_t>(2, 160 * 1024 / mm_tile_lds(t, nz, elem));
    const int64_t slots = 256 * (int64_t)per_cu, full = n / slots, rest = n - full * slots;
    return (elem == 8 ? 2.8 : 2.5) + one * (double)(full * per_cu + (rest + 255) / 256);
}

// ... and in the four stage kernels: their launches, then the traffic of meshes
// that the caches hold and of those that they don't (7 % and 9 % rms)
inline double mm_stage_us(double cells, int elem)
{
    if (elem == 8) return 21.0 + 7.8e-5 * std::min(cells, 4.5e5) + 1.2e-4 * std::max(cells - 4.5e5, 0.0);
    return 20.0 + 4.0e-5 * std::min(cells, 5e5) + 6.5e-5 * std::min(std::max(cells - 5e5, 0.0), 2.5e6) +
           7.2e-5 * std::max(cells - 3e6, 0.0);
}

// Tile width of the one-launch step for regions of nx0 (and nx1) x ny columns
// of nz cells, 0 for the stage kernels.  Among the tiles that fit, the one with
// the least (workgroups per CU, at least one) x (cells per thread): small meshes
// take small tiles (every CU busy), large ones the largest (least
// recomputation).  The stage kernels are taken where no tile fits and where their
// modelled time is 5 % or more below the tile's: tall meshes of many rounds, whose
// narrow tiles recompute 2 to 2.8 times their cells in every round (FP32
// 600x300x12 151 us a step against 224 in tiles, 1500x600x16 1025 against 2069;
// FP64 300x60x14 38.7 against 54.3, 420x200x12 117 against 196).  The choice is within
// 4 % of the faster one on all of the measured meshes but one (FP64 300x150x8: 51 in
// tiles, 48 in stages).
inline int mm_pick_tile(int nx0, int nx1, int ny, int nz, int elem)
{
    int pick = 0;
    int64_t pick_tiles = 0;
    double best = 1e300;
    for (int t : kMMTiles) {
        if (elem == 8 && t > kMMTileMax64) break;
        const int64_t nw = (int64_t)(t + 2 * kMMHalo) * (t + 2 * kMMHalo) * nz;
        if (nw > kMMThreads * kMMCells || mm_tile_lds(t, nz, elem) > kMMTileLds) continue;
        auto wide = [t](int n) { return ((int64_t)n + t - 1) / t; };
        const int64_t tiles = (wide(nx0) + wide(nx1)) * wide(ny);
        const double cost =
            std::max(1.0, (double)tiles / 256.0) * (double)((nw + kMMThreads - 1) / kMMThreads);
        if (cost < best) {
            best = cost;
            pick = t;
            pick_tiles = tiles;
        }
    }
    if (!pick) return 0;
    const double cells = ((double)nx0 + nx1) * ny * nz;
    return mm_stage_us(cells, elem) < 0.95 * mm_tile_us(pick, pick_tiles, nz, elem) ? 0 : pick;
}

}  // namespace asd
