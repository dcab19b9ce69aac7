// shape.h -- launch-shape rules of the host code: plain arithmetic without HIP,
// so that a host compiler alone can check them.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace rqa {

// One wavefront walks a band of TILE_W consecutive diagonals; lane L owns
// diagonal d0 + L and steps along it.
constexpr int TILE_W = 64;

// Most tiles of T steps that a chunk may hold.  The counting kernels count in
// 32-bit words and flush them between chunks only, so a chunk's cells have to
// fit: a caller's shape of 4096 tiles of 65,536 steps (2^34 cells) wrapped row
// sums of more than 2^32 - 1 cells.
constexpr uint32_t chunk_tiles_limit(uint32_t T) { return (uint32_t)(0xFFFFFFFFull / ((uint64_t)TILE_W * T)); }

// Tiles (band of TILE_W diagonals, segment of T steps) of a series whose longest
// diagonal, and number of diagonals, is L0: segment s holds B - s T / TILE_W
// bands.  Tiles are numbered in 31 bits.
constexpr uint64_t MAX_TILES = 1ull << 31;
inline uint64_t tile_count(uint64_t L0, uint32_t T)
{
    const uint64_t B = (L0 + TILE_W - 1) / TILE_W, S = (L0 + T - 1) / T, q = T / TILE_W;
    return S * B - q * (S * (S - 1) / 2);
}

// Default segment length when nothing is tuned, from the work of the whole call
// (pairs over all series) per wave of one 8-wave workgroup on every CU: a call
// with up to 512 steps for each gives each one tile, so that no CU waits for a
// second round of short tiles; a larger one about `tiles`, of 256 to 1024 steps.
// That is six, and nine for one series with a window selection, whose
// workgroups take sixteen tiles at a time: with six they take three or four times
// and the last time few of them find work (RR 80 .. 99 %, where that pass is most
// of the call, N = 40,000 and 48,000: 2.89 -> 2.46 and 3.89 -> 3.70 ms; RR 1 ..
// 20 %: 585 -> 545 and 720 -> 715 us; eleven and eighteen N = 1e4 series (m = 3)
// would lose: 560 -> 618 and 751 -> 783 us).
// Measured (us per call, K = 20, m = 1 unless said): one N = 1e4 series
// (381 steps) T = 128 / 256 / 512 / 1024: 233 / 181 / 175 / 231; twenty
// N = 3000 (686): 128 / 256 / 512: 339 / 289 / 326; N = 30,000 (3433): 128 /
// 512 / 1024: 549 / 510 / 547; the 600-series ensemble (87,000): 128 / 512 /
// 960: 6663 / 6331 / 5796.  From the walker's unit on (the two half-blocks of
// its ring and 64: 320 for m = 3, tau = 5, 192 for tau = 3, 64 else) a multiple
// of it, so that no segment ends with a part of a half-block, which takes the
// walker's edge path (two N = 1e5 series, tau = 5: 512 / 640: 5337 / 4787);
// but a series too long for that many tiles takes the 1024 it fits with.
inline uint32_t default_segment(uint64_t L0, uint64_t pairs, int num_cu, uint32_t unit, uint32_t tiles)
{
    const uint64_t steps = pairs / TILE_W / ((uint64_t)num_cu * 8);
    // an eighth more than its share, or a few workgroups would not find a CU
    if (steps <= 512) return (uint32_t)((steps * 9 / 8 + 63) / 64 * 64 + (steps ? 0 : 64));
    const uint32_t t = (uint32_t)std::min<uint64_t>(std::max<uint64_t>(steps / tiles, 256), 1024) / TILE_W * TILE_W;
    const uint32_t whole = t / unit * unit;
    return whole && tile_count(L0, whole) < MAX_TILES ? whole : t;
}

}  // namespace rqa
