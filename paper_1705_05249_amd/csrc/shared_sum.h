// How the sum of a shared-sum kernel (tiny.hip) is cut.  Plain host + device code, so that a host-side checker can walk every address.
#pragma once

#include <stdint.h>

#include "lds_layout.h"

namespace mg {

// Lines (values of k) at the end of an operand along its rows whose pieces are checked one by one.  A line is fetched in pieces of `piece` elements;
// the last one reaches `over` elements past the last row, into the lines behind it, and past the operand's end where these are too few: one
// line is enough but for operands of fewer than four rows, whose lines may be shorter than `over` (2 rows, ld 2: three; 1 row, ld 1: seven).
MG_HD constexpr int lines_kept_back(int64_t rows, int64_t ld, int piece)
{
    const int64_t over = (piece - rows % piece) % piece;
    return static_cast<int>((over + ld - 1) / ld);
}

// whole pairs of K-steps (`pair` values of k each) in a sum of k that keeps `kept` values back
MG_HD constexpr int whole_pairs(int k, int kept, int pair) { return k > kept ? (k - kept) / pair : 0; }

}  // namespace mg
