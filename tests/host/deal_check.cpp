// deal_tiles: every tile of a list is dealt exactly once, every XCD gets as many
// chunks, and the grid stays below half as many work-groups again.
#include <cstdio>
#include <vector>

#include "dwt2_internal.h"

int main() {
    int bad = 0;
    for (int64_t near : {2, 3, 10, 37, 64, 300, 4096})
        for (int64_t tiles : {1, 2, 7, 8, 9, 63, 64, 65, 511, 1023, 1024, 1025, 1083, 4095, 4096, 4097, 7585, 20011}) {
            const dwt2::Deal d = dwt2::deal_tiles(tiles, near);
            if (d.chunk < 1 || d.grid % (8 * d.chunk) || d.grid < tiles || d.grid > tiles + tiles / 2 + 8) ++bad;
            std::vector<int> seen(tiles, 0);
            for (int64_t b = 0; b < d.grid; ++b) {
                const int64_t j = b >> 3, n = ((j / d.chunk) * 8 + (b & 7)) * d.chunk + j % d.chunk;
                if (n < tiles) ++seen[n];
            }
            for (int c : seen) bad += c != 1;
        }
    const dwt2::Deal d = dwt2::deal_tiles(dwt2::kMaxTiles, 2);
    if (d.grid > 0x7fffffff || d.grid < dwt2::kMaxTiles) ++bad;
    std::printf("bad %d\n", bad);
    return bad != 0;
}
