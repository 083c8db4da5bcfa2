// The grid of a launch that takes one tile per workgroup, and how much of a
// tile exists.  Plain C++ without HIP headers, so that the arithmetic can also
// be run on the host, at sizes for which no buffer can be allocated.
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#define TC_HOST_DEVICE __host__ __device__
#else
#define TC_HOST_DEVICE
#endif

namespace tc {

struct GridXY {
    uint32_t x, y;
};

// Workgroups of `threads` for `tiles` tiles (at least one).  HIP takes fewer
// than 2^32 threads in one dimension, so past 2^31 the grid goes on along y,
// in whole rows: tile = y * grid.x + x, and the last row's workgroups past the
// last tile have nothing to do.
inline GridXY grid_of(int64_t tiles, int threads) {
    const int64_t most = (int64_t(1) << 31) / threads;
    if (tiles < 1) tiles = 1;
    if (tiles <= most) return GridXY{static_cast<uint32_t>(tiles), 1};
    return GridXY{static_cast<uint32_t>(most), static_cast<uint32_t>((tiles + most - 1) / most)};
}

// How many of the `total` items tile `tile` has, `per` to a full one: none in
// the tiles past the last.  Compared in 64 bits: the distance to those tiles
// does not fit 32 in a long last row.
TC_HOST_DEVICE inline int tile_items(int64_t total, int64_t tile, int per) {
    const int64_t left = total - tile * per;
    return left <= 0 ? 0 : left < per ? static_cast<int>(left) : per;
}

}  // namespace tc
