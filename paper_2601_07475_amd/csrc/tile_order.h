// Which tile of the output a workgroup computes, shared by the tiled GEMM kernels.
//
// Workgroups are dealt round-robin to the 8 XCDs, each with an L2 of its own.  Every XCD gets a contiguous run of the tile sequence
// (the first num_tiles % 8 of them one tile more), and the sequence walks groups of tile rows column by column, so that the 32 tiles
// an XCD computes at a time share their rows of A and W in that L2.
// Runs for tile counts that are multiples of 8 only, and the plain sequence for all others, cost the MXFP4 kernels, whose copies
// bind them, 4 % on average over 250 problems of 513 to 8192 rows (2387 x 8384 over K' = 2400, 13 x 33 tiles: 57.3 against 49.6 us;
// 1500 x 14336 over 4320: 89.5 against 82.5) and up to 28 %; the NVFP4 kernels 1 %.
#pragma once
#include <hip/hip_runtime.h>

namespace arcq {

// Tile rows of a group.  Computed on the host: a division less in front of a kernel's first copies.
// At most 8, about 8 x 4 tiles an XCD, in as few groups as that allows and about equal ones (17 rows 6, 6 and 5; 57 seven times 8 and
// one).  8 and what is left: 0.3 % slower; 6 or 4, or across columns first: 0.2 to 2 % slower.
// Tall problems go row by row: in groups, the run of an XCD ends in the middle of one, and with few columns it then reads the rows of two groups, while
// every XCD reads all of W anyway.  In MXFP4, 129 problems with 2 to 7 tile columns and 20 to 60 tile rows, us in groups and by rows: 1.04x on
// average, 1.06x from K' = 3000 on, 0.94 to 1.22x (6121 x 273 over K' = 8864 33.7 and 27.2, 5675 x 140 over 7072 26.6 and 21.7, 7533 x 395
// over 2208 11.2 and 11.4); NVFP4 1.015x over 45.  No clear gain any more with 8 to 11 columns, 1.01x (0.96 to 1.07), and with fewer than 20 rows,
// two and a half an XCD, 0.98 to 1.0x.
__host__ __device__ inline int tile_group_rows(int tiles_m, int tiles_n) {
    if (tiles_n < 8 && tiles_m >= 20) return 1;
    const int groups = (tiles_m + 7) / 8;
    return (tiles_m + groups - 1) / groups;
}

struct TileOrder {
    int m, n;       // tile row and column
    __host__ __device__ __forceinline__ TileOrder(int wg, int tiles_m, int tiles_n, int group_rows) {
        const int num_tiles = tiles_m * tiles_n;
        const int xcd = wg & 7, longer = num_tiles & 7;
        const int pid = xcd * (num_tiles >> 3) + (xcd < longer ? xcd : longer) + (wg >> 3);
        const int g = pid / (group_rows * tiles_n);
        const int first_m = g * group_rows, left = tiles_m - first_m;
        const int height = group_rows < left ? group_rows : left;
        const int in_g = pid - first_m * tiles_n;
        n = in_g / height;
        m = first_m + in_g - n * height;
    }
};

}  // namespace arcq
