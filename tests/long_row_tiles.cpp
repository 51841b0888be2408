// Host check of the long-row stages' tiles: for rows of 8193 to 2^23 elements and any batch a tile has 4608 to 16384 elements, a multiple of
// 512 (a wavefront's share of whole 64-element steps), the tiles cover the row, and there are at most 512 of them, 128 where they can be
// long enough in batches of up to 256 rows.  Ends with 1 at the first that does not hold.
#include <cmath>
#include <cstdio>

#include "../paper_2511_11608_amd/csrc/slicer_encode_large.hpp"

using namespace slicer;

int main()
{
    long n = 0;
    for (int64_t rows = 1; rows <= 65535; rows += rows < 1100 ? 1 : 4099)
        for (double len = 8193; len <= (1 << 23); len *= 1.013, ++n) {
            const int64_t N = (int64_t)len, tile = large_tile(rows, N), S = (N + tile - 1) / tile;
            if (tile % 512 || tile < 4608 || tile > 16384 || S > 512 || (S > 128 && rows <= 256 && N <= 128 * 16384)) {
                printf("[%lld x %lld]: %lld tiles of %lld\n", (long long)rows, (long long)N, (long long)S, (long long)tile);
                return 1;
            }
        }
    const int64_t longest = large_tile(1, 1 << 23);
    if (((1 << 23) + longest - 1) / longest > 512) return 1;
    printf("%ld shapes\n", n);
    return 0;
}
