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

// Division by a number known on the host: quot(q) = q / d for 0 <= q < 2^31, d >= 1.  (magic = ceil(2^shift / d) with
// 2^(shift - 31) >= d: the product is q / d * 2^shift and less than 2^shift / d too much.)  Three scalar instructions; what the
// compiler makes of a division by a kernel argument is some thirty behind a vector reciprocal.
struct Divisor {
    uint32_t d, magic;
    int shift;
    MG_HD inline uint32_t quot(uint32_t q) const { return static_cast<uint32_t>((static_cast<uint64_t>(q) * magic) >> shift); }
};
inline Divisor divisor(int64_t d)
{
    int shift = 31;
    while ((int64_t(1) << (shift - 31)) < d) ++shift;
    return Divisor{static_cast<uint32_t>(d), static_cast<uint32_t>(((uint64_t(1) << shift) + static_cast<uint64_t>(d) - 1) / static_cast<uint64_t>(d)), shift};
}

// Which tile of which instance a work-group takes.  Work-groups go to the eight XCDs in turn, and the tiles of an instance share
// its operands: of eight instances each XCD takes one, whose tiles lie eight work-groups apart and meet in its L2.  The last
// batch % 8 instances leave XCDs idle; where that is more than a sixth of the chip's time they are dealt out tile by tile,
// neighbours to the same XCD (us, undivided / dealt out: FP32 2048^3 one instance 1320 / 177, 1024^3 one 176 / 37, five 179 / 113; FP16
// 2048^3 one 249 / 44; 256^3 two, whose operands then come to eight L2s, 8.8 / 9.3).  Else they stay undivided too (FP16
// 7 x (300, 300, 40) 5.9 / 6.6, 118 x 91^3 7.5 / 7.9, 517 x (128, 128, 64) 12.2 / 12.6): a place past the last instance is an idle one.
struct Place {
    int64_t inst;
    uint32_t tile;
};
// (what a launch has in common is worked out on the host: instances of a few elements are over in a few hundred clocks)
struct Walk {
    Divisor tiles;                 // of an instance
    uint32_t sets;                 // whole sets of eight instances
    uint32_t undivided;            // work-groups that take a tile of an instance of their XCD; the others share the last instances:
    uint32_t share, more;          // each XCD has `share` of them, the first `more` XCDs one more
};
inline bool deals_out(int64_t batch) { return (8 - batch % 8) % 8 * 5 > batch; }
inline int64_t work_groups(int64_t batch, int64_t tiles) { return (deals_out(batch) ? batch : (batch + 7) / 8 * 8) * tiles; }
inline Walk walk(int64_t batch, int64_t tiles)
{
    const uint32_t t = static_cast<uint32_t>(tiles), sets = static_cast<uint32_t>(batch / 8), rest = static_cast<uint32_t>(batch % 8) * t;
    return Walk{divisor(tiles), sets, deals_out(batch) ? sets * 8 * t : ~0u, rest / 8, rest % 8};
}
MG_HD inline Place place(const Walk &w, uint32_t group)
{
    const uint32_t xcd = group % 8;
    uint32_t q = group / 8;
    const bool shared = group >= w.undivided;
    if (shared) q = xcd * w.share + (xcd < w.more ? xcd : w.more) + (q - w.sets * w.tiles.d);
    const uint32_t inst = w.tiles.quot(q);
    return Place{shared ? static_cast<int64_t>(w.sets) * 8 + inst : static_cast<int64_t>(inst) * 8 + xcd, q - inst * w.tiles.d};
}

// One launch has fewer than 2^32 threads, so at most this many work-groups of 256 (a multiple of eight keeps the XCDs in step)
constexpr int64_t MOST_GROUPS = (int64_t(1) << 24) - 8;

// The launches of a call: launch(first instance, instances, first tile, tiles of each instance) for every piece of it, until one
// returns false.  per_group: instances per work-group, 0: a work-group takes one tile of an instance.
template <typename Launch> inline bool for_pieces(int64_t batch, int64_t tiles, int64_t per_group, Launch launch)
{
    int64_t count = per_group > 0 ? MOST_GROUPS * per_group : (tiles < MOST_GROUPS ? MOST_GROUPS / tiles : 1);
    if (count >= 8) count -= count % 8;
    else if (per_group == 0 && tiles < MOST_GROUPS)
        while (work_groups(count, tiles) > MOST_GROUPS) --count;       // (idle places count)
    const int64_t most_tiles = per_group > 0 || tiles < MOST_GROUPS ? tiles : MOST_GROUPS;
    for (int64_t i = 0; i < batch; i += count)
        for (int64_t t = 0; t < tiles; t += most_tiles)
            if (!launch(i, batch - i < count ? batch - i : count, t, tiles - t < most_tiles ? tiles - t : most_tiles)) return false;
    return true;
}

}  // namespace batchwalk
}  // namespace mg
