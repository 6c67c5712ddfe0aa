// Reads lines "nx0 nx1 ny nz elem" and prints for each the tile width that the
// micromagnetic step takes (0: the stage kernels) and the LDS bytes of that tile.
#include <cstdio>

#include "asd_mm_tiles.h"

int main()
{
    int nx0, nx1, ny, nz, elem;
    while (std::scanf("%d %d %d %d %d", &nx0, &nx1, &ny, &nz, &elem) == 5) {
        const int t = asd::mm_pick_tile(nx0, nx1, ny, nz, elem);
        std::printf("%d %zu\n", t, t ? asd::mm_tile_lds(t, nz, elem) : (size_t)0);
    }
    return 0;
}
