// How the kernels of batched_tile.hip walk their work.  Plain host + device code, so that a host-side checker can run it at
// extents no test can afford on the device.
#pragma once

#include "lds_layout.h"

namespace mg {
namespace batchwalk {

// body(left) for each chunk of KC terms of a sum of k, left: the terms from this chunk on.  It counts what is left: the start of
// the chunk behind the last one would pass the largest int for k within KC of it, and the loop would not end.
template <int KC, typename Body> MG_HD inline void for_chunks(int k, Body body)
{
    for (int left = k; left > 0; left -= KC) body(left);
}

}  // namespace batchwalk
}  // namespace mg
