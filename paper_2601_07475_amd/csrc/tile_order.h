// Which tile of the output a workgroup computes, shared by the tiled GEMM kernels.
//
// Workgroups are dealt round-robin to the 8 XCDs, each with an L2 of its own.  Every XCD gets a contiguous run of the tile sequence
// (the first num_tiles % 8 of them one tile more), and the sequence walks groups of at most 8 tile rows (of equal height: the
// tile rows dealt out over as few groups as that allows) column by column, so that the 32 tiles an XCD computes at a time are
// about 8 x 4 and share their rows of A and W in that L2.
// Runs for tile counts that are multiples of 8 only, and the plain sequence for all others, cost the MXFP4 kernels, whose copies
// bind them, 4 % on average over 250 problems of 513 to 8192 rows (2387 x 8384 over K' = 2400, 13 x 33 tiles: 57.3 against 49.6 us;
// 1500 x 14336 over 4320: 89.5 against 82.5) and up to 28 %; the NVFP4 kernels 1 %.  Groups of 8 rows and what is left (one row of
// 17) instead of equal ones: 0.3 % slower; of 6 or 4, or across columns first: 0.2 to 2 % slower.  Tall problems of one round
// (17 x 13 tiles over K' = 14656: 138 us) run faster in the plain sequence, 127 us; on average over 12 such it is no better.
#pragma once
#include <hip/hip_runtime.h>

namespace arcq {

struct TileOrder {
    int m, n;       // tile row and column
    __device__ __forceinline__ TileOrder(int wg, int tiles_m, int tiles_n) {
        const int num_tiles = tiles_m * tiles_n;
        const int xcd = wg & 7;
        const int pid = xcd * (num_tiles >> 3) + min(xcd, num_tiles & 7) + (wg >> 3);
        const int groups = (tiles_m + 7) >> 3, rows = (tiles_m + groups - 1) / groups;
        const int g = pid / (rows * tiles_n);
        const int first_m = g * rows;
        const int height = min(rows, tiles_m - first_m);
        const int in_g = pid - first_m * tiles_n;
        m = first_m + in_g % height;
        n = in_g / height;
    }
};

}  // namespace arcq
