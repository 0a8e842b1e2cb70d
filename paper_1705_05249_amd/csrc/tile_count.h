// Tiles of a product whose C is a triangle.  Plain C++, so that a host-side checker can compile it.
#pragma once

#include <math.h>
#include <stdint.h>

#if defined(__HIPCC__)
#define MG_TILE_HD __host__ __device__
#else
#define MG_TILE_HD
#endif

namespace mg {

// Tile `id` of the tiles * (tiles + 1) / 2 square tiles that touch the lower triangle of C (the upper one's are their mirror image): groups of
// eight tile rows, column by column, so that tiles with ids close together share rows and columns.  A grid of all tiles hands
// the skipped ones out in turn with the others, and of 253 wanted tiles some compute units get two while others get none (FP16 SYRK 4096 on
// 192 x 192 tiles, all 484 / the wanted 253: 108 / 68 us).
MG_TILE_HD inline void triangle_tile(int id, int tiles, bool upper, int &tm, int &tn)
{
    constexpr int GROUP = 8;
    int g = static_cast<int>(sqrtf(static_cast<float>(id) * (1.f / 32.f)));
    // tiles in front of group g: 64 * (0 + ... + g - 1) + 36 g
    while (g > 0 && 4 * g * (8 * g + 1) > id) --g;
    while (4 * (g + 1) * (8 * (g + 1) + 1) <= id) ++g;
    const int first = g * GROUP, size = tiles - first < GROUP ? tiles - first : GROUP;
    int rest = id - 4 * g * (8 * g + 1), row, column;
    if (rest < size * first) {
        column = rest / size;
        row = first + rest % size;
    } else {                       // the triangle at the group's end: its column c has the rows from c on
        rest -= size * first;
        column = 0;
        while (rest >= size - column) rest -= size - column++;
        row = first + column + rest;
        column += first;
    }
    tm = upper ? column : row;
    tn = upper ? row : column;
}

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
