// Checks tl::tile_row_blocks (csrc/tl_grid.hpp): no grid reaches 2^32 threads, none is smaller than it has to be, and every row
// block is launched.
#include "tl_grid.hpp"

#include <cstdio>

int main()
{
    const int64_t limit = int64_t(1) << 32;
    for (int64_t tiles_n = 1; tiles_n <= int64_t(1) << 19; tiles_n += 1 + tiles_n / 97) {
        const int64_t blocks = tl::tile_row_blocks(tiles_n);
        if (blocks < 1 || blocks * tiles_n * tl::kTileThreads >= limit || (blocks + 1) * tiles_n * tl::kTileThreads < limit) {
            std::printf("tiles_n = %lld: %lld row blocks\n", (long long)tiles_n, (long long)blocks);
            return 1;
        }
    }
    // 262208 x 262208 in tiles of 64 x 128: the launch that wrapped
    const int64_t tiles_m = 4097, tiles_n = 2049, blocks = tl::tile_row_blocks(tiles_n);
    if (tiles_m * tiles_n * tl::kTileThreads < limit || blocks >= tiles_m || tiles_m - blocks > blocks) {
        std::printf("262208 x 262208: %lld of %lld row blocks\n", (long long)blocks, (long long)tiles_m);
        return 1;
    }
    std::puts("ok");
    return 0;
}
