// shape.h -- launch-shape rules of the host code: plain arithmetic without HIP,
// so that a host compiler alone can check them.
#pragma once

#include <stdint.h>

namespace rqa {

// One wavefront walks a band of TILE_W consecutive diagonals; lane L owns
// diagonal d0 + L and steps along it.
constexpr int TILE_W = 64;

// Most tiles of T steps that a chunk may hold.  The counting kernels count in
// 32-bit words and flush them between chunks only, so a chunk's cells have to
// fit: a caller's shape of 4096 tiles of 65,536 steps (2^34 cells) wrapped row
// sums of more than 2^32 - 1 cells.
constexpr uint32_t chunk_tiles_limit(uint32_t T) { return (uint32_t)(0xFFFFFFFFull / ((uint64_t)TILE_W * T)); }

}  // namespace rqa
