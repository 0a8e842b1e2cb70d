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

}  // namespace mg
