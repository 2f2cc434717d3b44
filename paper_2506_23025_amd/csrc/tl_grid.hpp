// How much of a matrix one launch of the tiled kernel covers (host side; plain C++, checked by a host program).
#pragma once
#include <cstdint>

namespace tl {

constexpr int64_t kTileThreads = 512;

// Row blocks of `tiles_n` tiles each that one grid holds: a launch counts its threads along x in 32 bits and takes a count that
// does not fit for what is left of it, without an error (64 x 128 tiles reach that at 137 GB of Y).  At least one: there
// are at most 2^24 columns.
inline int64_t tile_row_blocks(int64_t tiles_n)
{
    const int64_t tiles = ((int64_t(1) << 32) - 1) / kTileThreads;
    const int64_t blocks = tiles / tiles_n;
    return blocks > 0 ? blocks : 1;
}

}  // namespace tl
