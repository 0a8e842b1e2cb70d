// Tiles of a product whose C is a triangle.  Plain C++, so that a host-side checker can compile it.
#pragma once

#include <stdint.h>

namespace mg {

// How many of the across_m x across_n tiles of bm x bn entries touch the lower (i >= j) or the upper triangle of C: what the kernels
// do not skip.  bm is a multiple of bn, as in every tile of the table.  In closed form: counted tile column by tile column, for every
// tile that selection ranks, it took 170 us of host time at n = 2^20 and 1 us at 4096.
inline int64_t triangle_tiles(bool lower, int64_t across_m, int64_t across_n, int bm, int bn)
{
    const int64_t r = bm / bn;
    if (lower) {                       // column j has the rows from j / r on
        const int64_t columns = across_n < across_m * r ? across_n : across_m * r, q = columns / r, rest = columns % r;
        return columns * across_m - (r * (q * (q - 1) / 2) + rest * q);
    }
    const int64_t rows = across_m < (across_n + r - 1) / r ? across_m : (across_n + r - 1) / r;      // row i has the columns from r i on
    return rows * across_n - r * (rows * (rows - 1) / 2);
}

// Such a launch hands its work-groups to the eight dies in turn and each die to its four shader engines of eight compute units in turn, and
// tile_coords_balanced (mfma_kernel.h; groups of eight tile rows) says which tile each takes: the wanted tiles of the engine that gets most,
// times 32, i.e. what the launch costs as if evenly spread.  Work-groups that skip their tile count in the turns, so 15 x 30 tiles of 256 x 128,
// 240 of them wanted, leave one engine ten for its eight compute units, and 231 of 21 x 21 tiles nine.  `slices` of the sum are as many
// such grids one behind the other.
inline int64_t busiest_engine_tiles(bool lower, int64_t across_m, int64_t across_n, int bm, int bn, int slices)
{
    constexpr int64_t GROUP = 8;
    int64_t wanted[32] = {0}, wg = 0;
    for (int z = 0; z < slices; ++z)
        for (int64_t first = 0; first < across_m; first += GROUP) {
            const int64_t size = across_m - first < GROUP ? across_m - first : GROUP;
            const bool odd = (first / GROUP) % 2 != 0;
            int64_t shift = lower ? 0 : 1 % size;
            for (int64_t tn = 0; tn < across_n; ++tn) {
                for (int64_t r = 0; r < size; ++r, ++wg) {
                    int64_t row = (odd ? size - 1 - r : r) + shift;
                    if (row >= size) row -= size;
                    const int64_t m0 = (first + row) * bm, n0 = tn * bn;
                    wanted[wg % 32] += lower ? n0 < m0 + bm : m0 < n0 + bn;
                }
                if (++shift == size) shift = 0;
            }
        }
    int64_t most = 0;
    for (const int64_t w : wanted) most = w > most ? w : most;
    return 32 * most;
}

}  // namespace mg
