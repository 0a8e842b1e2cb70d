// How the kernels of batched_tile.hip walk their work.  Plain host + device code, so that a host-side checker can run it at
// extents no test can afford on the device.
#pragma once

#include <stdint.h>

#include "lds_layout.h"

namespace mg {
namespace batchwalk {

// body(left) for each chunk of KC terms of a sum of k, left: the terms from this chunk on.  It counts what is left: the start of
// the chunk behind the last one would pass the largest int for k within KC of it, and the loop would not end.
template <int KC, typename Body> MG_HD inline void for_chunks(int k, Body body)
{
    for (int left = k; left > 0; left -= KC) body(left);
}

// Which tile of which instance a work-group takes.  Work-groups go to the eight XCDs in turn, and the tiles of an instance share
// its operands: of eight instances each XCD takes one, whose tiles lie eight work-groups apart and meet in its L2.  Of fewer
// than 128 instances the last batch % 8 are dealt out tile by tile, neighbours to the same XCD: one instance alone would
// otherwise keep one XCD busy and seven idle (us, undivided / dealt out: FP32 2048^3 one instance 1320 / 177, 1024^3 one 176 / 37,
// five 179 / 113; FP16 2048^3 one 249 / 44; 256^3 two, whose operands then come to eight L2s, 8.8 / 9.3).  Of more instances
// the last ones stay undivided too (517 x (128, 128, 64) FP16 12.2 / 12.6): a place past the last instance is an idle one.
struct Place {
    int64_t inst;
    uint32_t tile;
};
MG_HD inline bool deals_out(int64_t batch) { return batch < 128; }
MG_HD inline int64_t work_groups(int64_t batch, int64_t tiles) { return (deals_out(batch) ? batch : (batch + 7) / 8 * 8) * tiles; }
MG_HD inline Place place(uint32_t group, int64_t batch, uint32_t tiles)
{
    const uint32_t sets = static_cast<uint32_t>(batch / 8), rest = static_cast<uint32_t>(batch % 8) * tiles;
    const uint32_t xcd = group % 8, share = rest / 8, more = rest % 8;
    const bool undivided = !deals_out(batch) || group < sets * 8 * tiles;
    const uint32_t q = undivided ? group / 8 : xcd * share + (xcd < more ? xcd : more) + (group / 8 - sets * tiles), inst = q / tiles;
    return Place{undivided ? static_cast<int64_t>(inst) * 8 + xcd : static_cast<int64_t>(sets) * 8 + inst, q - inst * tiles};
}

// One launch has fewer than 2^32 threads, so at most this many work-groups of 256 (a multiple of eight keeps the XCDs in step)
constexpr int64_t MOST_GROUPS = (int64_t(1) << 24) - 8;

// The launches of a call: launch(first instance, instances, first tile, tiles of each instance) for every piece of it, until one
// returns false.  per_group: instances per work-group, 0: a work-group takes one tile of an instance.
template <typename Launch> inline bool for_pieces(int64_t batch, int64_t tiles, int64_t per_group, Launch launch)
{
    int64_t count = per_group > 0 ? MOST_GROUPS * per_group : (tiles < MOST_GROUPS ? MOST_GROUPS / tiles : 1);
    if (count >= 8) count -= count % 8;
    const int64_t most_tiles = per_group > 0 || tiles < MOST_GROUPS ? tiles : MOST_GROUPS;
    for (int64_t i = 0; i < batch; i += count)
        for (int64_t t = 0; t < tiles; t += most_tiles)
            if (!launch(i, batch - i < count ? batch - i : count, t, tiles - t < most_tiles ? tiles - t : most_tiles)) return false;
    return true;
}

}  // namespace batchwalk
}  // namespace mg
