#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <string_view>
#include <unordered_map>

#include "select.h"
#include "tile_count.h"

namespace mg {
namespace {

// (an index of the one, fixed table: comparing names one by one was half of a selection's time, 0.3-0.5 us of a call)
int32_t find(const std::vector<KernelEntry> &table, const char *name)
{
    static const std::unordered_map<std::string_view, int32_t> ids = [&table] {
        std::unordered_map<std::string_view, int32_t> m;
        for (size_t i = 0; i < table.size(); ++i) m.emplace(table[i].name, static_cast<int32_t>(i));
        return m;
    }();
    const auto it = ids.find(name);
    return it == ids.end() ? -1 : it->second;
}

bool try_pick(const std::vector<KernelEntry> &table, const Problem &p, int64_t alignment, const char *name,
              int split, int32_t *kernel, int32_t *out_split)
{
    const int32_t id = find(table, name);
    if (id < 0 || !table[id].legal || !table[id].legal(p, split, alignment)) return false;
    *kernel = id;
    *out_split = split;
    return true;
}

// MFMA kernel of tile `tag` for this problem's operand contiguity: the fast flavour if the problem
// is aligned and made of whole tiles, else the edge flavour.
bool try_mfma(const std::vector<KernelEntry> &table, const Problem &p, int64_t alignment, const char *tag, int split,
              int32_t *kernel, int32_t *out_split)
{
    char name[96];
    const char *contig = p.a_trans ? (p.b_trans ? "kn" : "kk") : (p.b_trans ? "mn" : "mk");
    // operands padded to whole tiles and the caller's own C (Problem::clip_m, clip_n): the direct-to-LDS kernels have a
    // flavour whose epilogue checks bounds, nothing else has
    if (p.clip_m != 0 || p.clip_n != 0) {
        if (strcmp(tag, "hdma16_256x256x64_w2x4") == 0)
            snprintf(name, sizeof name, "%s_256x256x64_w2x4_%s", p.b_trans ? "hdma16c" : "hpp16c", contig);
        else if (strcmp(tag, "hdma16_128x128x64_w2x4") == 0)
            snprintf(name, sizeof name, "hdma16c_128x128x64_w2x4_%s", contig);
        else if (strcmp(tag, "hdma16_256x128x64_w4x2") == 0)
            snprintf(name, sizeof name, "hdma16c_256x128x64_w4x2_%s", contig);
        else if (strcmp(tag, "hdeep16_128x128x64_w2x4") == 0)
            snprintf(name, sizeof name, "hdma16c_deep_128x128x64_w2x4_%s", contig);
        else
            return false;
        return try_pick(table, p, alignment, name, split, kernel, out_split);
    }
    // with B contiguous along k the 256 x 256 direct-to-LDS tile has a faster schedule (wavefronts taking turns:
    // 4096^3 102 -> 99 us, 8192^3 820 -> 747 us, 2048^3 42 -> 38 us)
    if (!p.b_trans && strcmp(tag, "hdma16_256x256x64_w2x4") == 0) {
        snprintf(name, sizeof name, "hpp16_256x256x64_w2x4_%s", contig);
        if (try_pick(table, p, alignment, name, split, kernel, out_split)) return true;
    }
    snprintf(name, sizeof name, "%s_%s", tag, contig);
    if (try_pick(table, p, alignment, name, split, kernel, out_split)) return true;
    // the register-staged 256 x 256 tile has its bounds-checked flavour on eight wavefronts only (on four, 256
    // accumulators per lane leave the checked loads no registers).  Ragged FP16 cubes in place, us, this flavour /
    // the best smaller tile: 3000 66-94 / 91-94, 5002 255-308 / 342-357, 4104 198-248 / 200-202, 2050 52-67 / 38-43
    // (the estimate below ranks all four the right way round)
    if (strcmp(tag, "hmfma_256x256x64_w2x2") == 0) tag = "hmfma_256x256x64_w2x4";
    snprintf(name, sizeof name, "%s_%s_edge", tag, contig);
    return try_pick(table, p, alignment, name, split, kernel, out_split);
}

struct TileChoice {
    const char *tag;
    int bm, bn, bk;
    float ceiling;       // Mflop/us per compute unit with enough resident work-groups
    float per_group;     // ... contributed by each resident work-group
    int resident;        // work-groups a compute unit holds at once
};

constexpr int kComputeUnits = 256;

// Split-K factor for a grid of `blocks` work-groups that each walk `ktiles` K-tiles.  From the sweep:
// a handful of blocks should be split until every compute unit has two (when K has >= 16 tiles and each
// slice keeps >= 4 of them); a grid that fills the chip less than four times over gains from splitting only when K
// is long (each slice keeps >= 24 K-tiles), because the reduce pass costs a launch and a round trip of
// the partial sums; otherwise no split.
int pick_split(int64_t blocks, int64_t ktiles)
{
    int64_t split = 1;
    if (blocks <= 64 && ktiles >= 16) {
        split = ceil_div(2 * kComputeUnits, blocks);
        if (split > ktiles / 4) split = ktiles / 4;
    } else if (blocks < 4 * kComputeUnits && ktiles >= 48) {
        split = ceil_div(4 * kComputeUnits, blocks);
        if (split > ktiles / 24) split = ktiles / 24;
    }
    if (split > 16) split = 16;
    return split < 1 ? 1 : static_cast<int>(split);
}

// Slices of the sum for a matrix-vector product.  Measured: the axpy kernel (32 KB of loads in flight per
// work-group) is fastest with about two work-groups per compute unit, the dot kernel (16 KB) with four; more
// gain nothing and the reduce pass costs.  Each slice keeps at least four rounds of loads, and the partial
// sums must fit the workspace.
constexpr int64_t kMostGemvSlices = 256;         // what the matrix-vector kernels take
int pick_gemv_split(const mg_config &cfg, int64_t outputs, int64_t k, size_t workspace_bytes)
{
    const bool dot = cfg.lds_bytes == 0;
    const int64_t wanted = (dot ? 4 : 2) * kComputeUnits;
    const int64_t groups = ceil_div(outputs, cfg.tile_m);
    if (2 * groups > wanted) return 1;
    // (the axpy kernel rounds down: a few work-groups more than two per compute unit take a third turn of their own; us, up / down:
    // 3072 x 16384 37.8 / 33.5, 9000^2 62.8 / 54.1, FP16 24576 x 7680 71.7 / 60.5, 60000 x 3000 69.2 / 60.4)
    int64_t split = dot ? ceil_div(wanted, groups) : wanted / groups;
    if (split > k / (4 * cfg.tile_k)) split = k / (4 * cfg.tile_k);
    if (split > kMostGemvSlices) split = kMostGemvSlices;
    const int64_t fits = static_cast<int64_t>(workspace_bytes / (static_cast<size_t>(outputs) * sizeof(float)));
    if (split > fits) split = fits;
    return split < 1 ? 1 : static_cast<int>(split);
}

// Matrix-vector product whose matrix lies along the outputs: the kernel and its slices.  us, FP32 unless said, axpy kernel (with
// its slices) / panel kernel:
//   a sum of at most 2560 terms (4224 where the columns do not lie a multiple of 4 KB apart) needs no second launch: 1024^2
//   11.7 / 8.2, 2048^2 11.3 / 9.7, 6144 x 3072 15.0 / 14.0, 4160 x 4096 14.3 / 11.7, FP16 11.8 / 9.2 (3072 x 6144 unsliced: 17.7);
//   else one work-group of sixteen wavefronts per compute unit: 4096^2 20.8 / 13.1, 4097 x 4095 16.7 / 14.2, 1024 x 16384
//   14.7 / 13.0, FP16 4096^2 11.7 / 10.8;
//   matrices beyond 96 MB, which stream from memory, stay with the axpy kernel: 7000^2 35.0 / 35.2, 10000^2 65.7 / 73.7,
//   65536 x 1024 41 / 44, 512 x 97656 35.0 / 42.6, 16384 x 4608 49.9 / 56.6, FP16 1024 x 97656 39.7 / 46.0.  Up to 384 MB
//   and with columns a multiple of 4 KB apart there are three exceptions, with four work-groups of the panel kernel per
//   compute unit: the columns are a power of two apart and the axpy kernel's slices a multiple of 2 MB (they meet on the
//   same channels; 8192^2 55.2 / 49.5, 4096 x 8192 33.1 / 25.6, 2048 x 16384 35.8 / 27.2, FP16 16384 x 4096 31.0 / 26.7;
//   beside them 8192 x 8200 44.5 / 49.4 and 6144 x 10240 42.9 / 44.5), with neither few work-groups of it along the outputs
//   (1024 x 65536 44.1 / 46.2, 192 x 260416 33.4 / 43.7) nor one of the panel kernel per compute unit (16384 x 4096 48.7 /
//   52.3); the outputs leave most lanes of an axpy work-group idle (64 x 390625 36.2 / 20.6, FP16 256 x 390625 54.9 / 37.7;
//   128 x 390625 38.9 / 37.9, FP16 512 x 195312 40.1 / 43.9); or they end inside a lane's run (about even: FP16 1500 x 66666
//   33.8 / 37.3, 9001 x 8000 28.7 / 25.4, 6001 x 9000 25.8 / 20.1, FP32 3001 x 12000 24.9 / 25.2, 14001 x 4001 35.7 / 39.6);
//   the axpy kernel also where its work-groups fill the chip by themselves (10^6 x 64: 40 / 66).
void pick_gemv_along_outputs(const std::vector<KernelEntry> &table, const Problem &p, int64_t alignment, size_t workspace_bytes,
                             int32_t *kernel, int32_t *split)
{
    const bool f32 = p.dtype == MG_F32;
    const int64_t outputs = p.m * p.n, lane_elems = 16 / static_cast<int64_t>(p.elem());
    const double bytes = static_cast<double>(outputs) * static_cast<double>(p.k) * static_cast<double>(p.elem());
    const int64_t stride = (p.n == 1 ? p.a_sk() : p.b_sk()) * static_cast<int64_t>(p.elem());
    const char *axpy = f32 ? "gemv_axpy_f32" : "gemv_axpy_f16";
    const bool streams = bytes > 96.0e6;
    const int64_t fits = static_cast<int64_t>(workspace_bytes / (static_cast<size_t>(outputs) * sizeof(float)));
    bool by_axpy = bytes > 384.0e6 || (streams && (p.k <= 2560 || stride % 4096 != 0)) || outputs >= 64 * lane_elems * kComputeUnits;
    if (streams && !by_axpy) {
        const mg_config &cfg = table[find(table, axpy)].cfg;
        const int slices = pick_gemv_split(cfg, outputs, p.k, ~size_t(0));
        const bool collide = (stride & (stride - 1)) == 0 && ceil_div(ceil_div(p.k, slices), cfg.tile_k) * cfg.tile_k * stride % (int64_t(2) << 20) == 0 &&
                             outputs >= 8 * cfg.tile_m && outputs < 16 * lane_elems * kComputeUnits;
        by_axpy = !(collide || outputs <= (f32 ? 64 : 256) || outputs % lane_elems != 0);
    }
    // A sum of a few terms is over before sixteen wavefronts have met (us, axpy / panel with 16 lanes: 1000 x 4 2.1 / 2.3, 16384 x 16
    // 2.4 / 2.6, 40000 x 32 3.1 / 3.8, 65472 x 32 3.1 / 4.4, FP16 65472 x 32 3.3 / 3.9; 16384 x 64 3.6 / 2.7), and where FP32 panels
    // would be three or more work-groups a compute unit (40000 x 64 4.0 / 4.4, 65472 x 128 7.1 / 7.7, x 192 9.4 / 9.6; FP16 x 64 4.3 /
    // 4.0).  Not where the outputs end inside a lane's run: there (tight columns, which start off 16 bytes) FP32 sums of 33 to 128 terms
    // take 1.3 times the panels' time (20 of 20 slower, 53963 x 126 9.3 / 6.5), and shorter ones go either way (65535 x 32 4.7 / 5.4, 9494 x 31
    // 4.2 / 3.5, FP16 68847 x 12 3.6 / 5.7, 42201 x 23 5.6 / 4.7).
    const bool even = outputs % lane_elems == 0;
    if (p.k <= 8 || (even && (p.k <= 32 || (f32 && p.k <= 128 && outputs > 32768)))) by_axpy = true;
    if (by_axpy) {
        if (!try_pick(table, p, alignment, axpy, 1, kernel, split)) return;
        const int want = pick_gemv_split(table[*kernel].cfg, outputs, p.k, workspace_bytes);
        if (want > 1) try_pick(table, p, alignment, axpy, want, kernel, split);
        return;
    }
    auto panel = [&](int lanes, int slices) {
        char name[32];
        snprintf(name, sizeof name, "gemv_panel%d_%s", lanes, f32 ? "f32" : "f16");
        return try_pick(table, p, alignment, name, slices, kernel, split);
    };
    if (p.k > 2560 && !(p.k <= 4224 && stride % 4096 != 0 && outputs >= 64 * 8 * lane_elems)) {
        const int64_t groups = ceil_div(outputs, 16 * lane_elems);
        // (rounded down: one work-group more than the compute units doubles the time of one of them; us, up / down: 1500 x 12000
        // 17.2 / 15.9, FP16 3000 x 12000 17.9 / 16.5, 5000 x 8192 18.4 / 17.4)
        int64_t slices = (streams ? 4 : 1) * kComputeUnits / groups;
        if (slices > p.k / 512) slices = p.k / 512;             // one round of a work-group's loads per slice
        if (slices > kMostGemvSlices) slices = kMostGemvSlices;
        if (slices > fits) slices = fits;
        if (slices > 1 && panel(16, static_cast<int>(slices))) return;
    }
    // Unsliced: the fewest lanes on a column that leave no compute unit a second work-group (us, FP32, 4 lanes / 8: 2048 x 4096 with
    // an odd leading dimension 10.2 / 12.6, 3000 x 4224 11.2 / 14.0, 4000 x 4224 12.4 / 11.8; 8 lanes / 16: 8192 x 2000 12.4 /
    // 12.7, 9000 x 2560 23.3 / 16.9, FP16 18000 x 2560 24.1 / 17.7).  With more outputs, and so a shorter sum, sixteen (8 / 16:
    // 20000 x 256 6.3 / 5.7, 40000 x 512 13.7 / 13.0, FP16 60000 x 512 13.0 / 10.6), but eight for FP32 sums beyond 256 up to 32768
    // outputs (20000 x 700 10.2 / 10.7, 32768 x 512 11.7 / 13.0) and where FP16 columns do not start on 16 bytes (65535 x 384
    // 15.2 / 17.3).  Sums of at most 128 terms leave half of the wavefronts of eight lanes without a column: sixteen (4 / 8 /
    // 16: 4096 x 64 2.9 / 2.7 / 2.5, 32768 x 64 8.7 / 5.1 / 3.1).
    const int64_t one_lane = lane_elems * kComputeUnits;        // outputs of a work-group per compute unit, per lane on a column
    if (p.k <= 128) panel(16, 1);
    else if (outputs <= 3 * one_lane) panel(4, 1);
    else if (outputs <= 8 * one_lane) panel(8, 1);
    else if (outputs <= 16 * one_lane || p.k <= 256) panel(16, 1);
    else panel(outputs > 32768 && (f32 || stride % 16 == 0) ? 16 : 8, 1);
}

// Longest sum that FP32 products of `blocks32` 32 x 32 blocks share among a block's wavefronts.  (Both operands along k, up to 64 blocks: 0.94 up to 1280 terms, 1.05 to 1.15
// up to 1792, 15 of 16 slower.  Behind the unfold pass, 51 layers of 1281 to 2048 terms: up to 64 blocks 1.08 up to 1536 terms, more 0.98 up to 1536, 0.98
// with two of nine up to 1.11 beyond; where there is room for slices)
int64_t most_shared_f32(const Problem &p, int64_t blocks32, bool unfolded)
{
    if (blocks32 > 64) return unfolded ? 1536 : 2048;
    return unfolded || (p.a_trans && !p.b_trans) ? 1280 : 1536;
}

}  // namespace

bool shared_without_fringe(const Problem &p)
{
    const int64_t blocks32 = ceil_div(p.m, 32) * ceil_div(p.n, 32);
    return blocks32 <= kComputeUnits && p.k <= 1024;
}

void select_config(const std::vector<KernelEntry> &table, const Problem &p, int64_t alignment, size_t workspace_bytes,
                   int32_t *kernel, int32_t *split, double *estimated_us)
{
    if (estimated_us != nullptr) *estimated_us = 0.0;
    *kernel = -1;
    *split = 1;
    const bool f32 = p.dtype == MG_F32;
    if (p.alpha == 0.f || p.k == 0) {
        try_pick(table, p, alignment, f32 ? "scale_f32" : "scale_f16", 1, kernel, split);
        return;
    }
    if (p.m == 1 || p.n == 1) {
        // short rows, thousands of them: four rows per wavefront keep enough loads in flight (long rows a power
        // of two apart are slower that way than one by one)
        const bool many = p.m * p.n >= 16 * kComputeUnits && p.k * static_cast<int64_t>(p.elem()) <= 4096;
        const char *dot = f32 ? (many ? "gemv_dot4_f32" : "gemv_dot_f32") : (many ? "gemv_dot4_f16" : "gemv_dot_f16");
        if (try_pick(table, p, alignment, dot, 1, kernel, split)) {
            const int want = pick_gemv_split(table[*kernel].cfg, p.m * p.n, p.k, workspace_bytes);
            if (want > 1) try_pick(table, p, alignment, dot, want, kernel, split);
        } else {
            pick_gemv_along_outputs(table, p, alignment, workspace_bytes, kernel, split);
        }
        if (*kernel >= 0) return;
    }
    // Problems of at most one 32 x 32 block per compute unit: the kernel whose eight wavefronts share the sum of one block (tiny.hip) beats the
    // macro tiles' software pipeline, which never fills, and saves the second launch of a sliced sum, until its eight shares grow longer
    // than those of slices.  Its time over that of the best macro tile with any slices, geometric means over 260 problems of up to 256 blocks in
    // all orders: FP32 of up to 128 terms 0.75, 256 0.62, 512 0.61, 768 0.69, 1024 0.80, 1536 0.90 (2048 1.12 on up to 64 blocks, 0.84 on
    // more; 2560 1.10); FP16 0.98 up to 256, 512 0.94, 768 0.85, 1024 0.78, 1536 0.82, 2048 0.81, 2560 0.84 (3072 0.93, 4096 0.94, beyond
    // 1.2), where the time of ranking the tiles, 0.5 us, comes on top.  More blocks than compute units: 1.2 to 1.8.
    // (with fringe rows / columns taken off, the tiles cover tm x tn of C)
    const int64_t tm = p.m - p.fringe_m, tn = p.n - p.fringe_n;
    // (of a triangle of C the blocks that touch it)
    const bool triangular_c = p.shape == MG_SHAPE_C_LOWER || p.shape == MG_SHAPE_C_UPPER;
    const int64_t blocks32 = triangular_c ? ceil_div(p.m, 32) * (ceil_div(p.m, 32) + 1) / 2 : ceil_div(p.m, 32) * ceil_div(p.n, 32);
    const char *order_tag = p.a_trans ? (p.b_trans ? "kn" : "kk") : (p.b_trans ? "mn" : "mk");
    const bool few_blocks = !p.tiles_only && blocks32 <= kComputeUnits && p.m > 1 && p.n > 1;
    // FP16 products of whole 64 x 64 tiles (aligned operands) and few K-tiles of 64 are ranked with the tiles, below: the register-staged ones without
    // checks start their products after one load, five work-groups to a compute unit.
    const bool whole64 = !f32 && p.conv == nullptr && p.m % 64 == 0 && p.n % 64 == 0 && p.k % 64 == 0 && dma_ragged_operands(p, alignment);
    const bool whole_short = whole64 && p.shape == MG_SHAPE_GENERAL && (p.k <= 256 || (p.k <= 384 && p.m / 64 * (p.n / 64) <= kComputeUnits));
    // (of a triangle of C they always are: over 123 SYRK of up to four K-tiles 64 x 64 ones take 0.93 of the time of what was chosen before the direct-to-LDS tiles
    // for any size, at most 1.01, and within 1 % of the fastest of all; (640, 64) 4.1 us, 4.5 on those tiles)
    if (triangular_c && whole64 && p.k <= 256) {
        char name[48];
        snprintf(name, sizeof name, "hmfma_64x64x64_w2x2_%s", order_tag);
        if (try_pick(table, p, alignment, name, 1, kernel, split)) return;
    }
    const int64_t most_f32 = most_shared_f32(p, blocks32, p.unfolded && p.m >= 16 && p.n >= 16 && workspace_bytes / 8 >= static_cast<size_t>(p.m) * static_cast<size_t>(p.n));
    // (FP16 on 1500 aligned products: neither operand along k, which the tiles read by transposing loads as well, its time over that of the tiles 1.06 to 1.12 up to 640 terms, 250 of
    // 275 slower, 0.96 from there to 1024; other orders 1.0 down to 0.85 from 65 to 640)
    const bool aligned16 = !f32 && dma_ragged_operands(p, alignment) && dma_offsets_fit(p, 192, 64);
    // (FP16 products with a triangular operand, whose sums are half as long: on tiles / here up to 64 terms 54 calls 1.07 times as long, to 128 1.04, to 256 1.02, to 512
    // 0.92, to 1024 0.82; (64, 64) 8.1 / 8.5 us with the copies in front; thin ones have no better kernel below)
    const bool short_triangle_operand = !f32 && p.shape != MG_SHAPE_GENERAL && !triangular_c && p.m >= 16 && p.n >= 16;
    const int64_t least = aligned16 && !p.a_trans && p.b_trans ? 641 : (short_triangle_operand ? 129 : 48), most = f32 ? most_f32 : 2560;
    if (few_blocks && !whole_short && p.k >= least && p.k <= most) {
        char name[48];
        snprintf(name, sizeof name, "%ctiny_32x32_%s", f32 ? 's' : 'h', order_tag);
        if (try_pick(table, p, alignment, name, 1, kernel, split)) return;
    }
    // Thin products (fewer than 16 rows or columns) beyond the shared-sum kernel's range are ranked like the others: most of a tile is empty, but the kernel
    // below, for any problem, loads element by element and does not slice its sums (us, that kernel / ranked: FP16 8 x 5416 x 4000 755 / 16, 13 x 1381 x 6016
    // 909 / 12, FP32 8 x 576 x 4952 530 / 15, 8 x 24720 x 8040 1455 / 211, 28481 x 12 x 621 94 / 27; sums of up to 48 terms stay on it).
    const bool thin = (p.m < 16 || p.n < 16) && p.m > 1 && p.n > 1 && p.k > 48;
    if ((p.m >= 16 && p.n >= 16) || thin) {
        // The macro tile (and number of K slices) with the smallest estimated time, see `estimate` below: a chip
        // that is not full runs ceil(tiles / 256) work-groups per compute unit at a rate that grows with them up to
        // the kernel's ceiling; a full chip works through rounds of 256 x resident work-groups.  Rates (Mflop/us per
        // compute unit: ceiling, per resident work-group) and the number of resident work-groups are fitted to a
        // scan of every tile over problems of 256 to 4608 tiles in the four operand orders, less 2.5 us per launch
        // (what a run of any length costs on top; common to all candidates, so not part of the estimate); partial
        // tiles of ragged problems count as whole ones.  The direct-to-LDS kernels need whole tiles and 16-byte aligned
        // operands; where they are illegal the next best estimate is tried.
        static const TileChoice f16_tiles[] = {{"hdma16_256x256x64_w2x4", 256, 256, 64, 4.88f, 4.83f, 1},
                                               {"hdma16_256x128x64_w4x2", 256, 128, 64, 4.4f, 4.3f, 1},
                                               {"hdma16_128x128x64_w2x4", 128, 128, 64, 4.07f, 2.75f, 2},
                                               {"hmfma_256x256x64_w2x2", 256, 256, 64, 4.54f, 4.40f, 1},
                                               {"hmfma_256x128x64_w2x2", 256, 128, 64, 3.72f, 3.72f, 1},
                                               {"hmfma_128x128x64_w2x2", 128, 128, 64, 3.61f, 3.0f, 2},
                                               {"hmfma_128x64x64_w2x2", 128, 64, 64, 2.85f, 1.87f, 3},
                                               {"hmfma_64x64x64_w2x2", 64, 64, 64, 2.30f, 1.65f, 5},
                                               {"hdeep16_128x128x64_w2x4", 128, 128, 64, 4.0f, 4.0f, 1},
                                               {"hdma16r_192x192x64_w2x4", 192, 192, 64, 0.f, 0.f, 1},
                                               {"hdma16r_192x128x64_w2x4", 192, 128, 64, 0.f, 0.f, 1},
                                               {"hdma16r_128x128x64_w2x4", 128, 128, 64, 0.f, 0.f, 1},
                                               {"hdma16r_128x64x64_w4x2", 128, 64, 64, 0.f, 0.f, 1},
                                               {"hdma16r_64x64x64_w2x2", 64, 64, 64, 0.f, 0.f, 2}};
        constexpr int kDeep = 8;            // index of the one with four stages
        constexpr int kRagged = 9, kRaggedSmallest = 13;      // indices of the direct-to-LDS kernels for sizes that end inside a tile
        // Their time in us, fitted to every tile with 1 to 8 slices on 310 sizes of 64 to 6000 in the four operand orders (residuals 5 to 8 %
        // rms): turns of one tile per compute unit, each a fixed part and, per K-tile, a part that grows with the square of the share of
        // the chip that is busy (the power limit) and the part of a second resident work-group; both operands along k / neither / A along m and B
        // along k; rows of an operand along k that are no multiple of 128 bytes apart (each 128-byte piece of a row touches two
        // lines); the traffic of C and of the partial sums.
        struct RaggedCost {
            double turn, ktile, ktile_load, second, both_k, neither_k, one_k, stray_rows, c, sums;
        };
        static const RaggedCost ragged_costs[5] = {{2.5, 0.607, 0.283, 0.0, 0.95, 1.05, 1.01, 0.08, 0.59, 0.86},
                                                   {2.1, 0.442, 0.237, 0.0, 0.94, 1.09, 1.04, 0.10, 0.69, 0.95},
                                                   {1.0, 0.308, 0.180, 0.0, 0.96, 1.11, 1.06, 0.12, 1.14, 0.99},
                                                   {1.2, 0.205, 0.116, 0.0, 0.94, 1.13, 1.04, 0.12, 0.84, 0.82},
                                                   {1.2, 0.163, 0.025, 0.179, 0.95, 1.12, 1.05, 0.12, 0.49, 0.64}};
        // Of sums of up to four K-tiles these are up to 40 % off, since a turn is then its first load and its epilogue, and the register-staged
        // kernels have their place: whole tiles, and checked ones for several turns of single K-tiles ((560, 6952, 64) with
        // beta 64 x 64 7.2 us, 64 x 64 / 128 x 128 direct-to-LDS 9.1 / 10.5).  Their times in us, fitted to 820 sizes of 64 to 8192 (the checked tiles' to those of
        // more than one turn) and to 670 whole ones, 3 to 6 % rms: a fixed part; turns of one tile per compute unit; and what a busier chip takes longer.
        // Fitted to half of the sizes and chosen for the other half, against the kernels without the direct-to-LDS tiles for any size: 0.886 of the time
        // (whole ones 0.98), 16 of 777 (9 of 334) more than 3 % slower, at most 10 % (19 %); by the costs above 0.907 (1.03), 91 (147), up to 28 % (43 %).
        struct ShortCost {
            double fixed, turn, turn_beta, ktile, busy, fixed_beta = 0.0, busy_beta = 0.0;
        };
        // general products | of whole tiles | triangles of C (400 sizes of 64 to 6200; 5 of 204 held out more than 3 % slower, without 16, up to 29 %;
        // (4416, 120) with beta 24.5 us on 64 x 64 direct-to-LDS tiles, 18.6)
        // | general products with beta whose rows of C end inside a 16-byte piece, which the large tiles fetch element by element: (4391, 1435, 128) 192 x 192 23.3 us, checked 64 x 64 12.7.
        // Fitted to half of 1560 such products, on the other half 1.007 times the best tile (by the first row 1.051), 60 instead of 224 of 782 more than 3 % slower, at most
        // 1.32 instead of 1.81 times
        static const ShortCost short_costs[4][14] = {{{}, {}, {}, {}, {}, {},
                                                      {3.61, 0.45, 0.48, 0.26, 0.88},
                                                      {3.50, 0.20, 0.21, 0.15, 0.56},
                                                      {},
                                                      {2.41, 3.02, 2.12, 0.65, 2.88},
                                                      {2.03, 3.21, 1.51, 0.50, 1.85},
                                                      {1.84, 2.42, 1.06, 0.37, 1.28},
                                                      {1.66, 1.92, 0.54, 0.27, 0.68},
                                                      {2.62, 0.72, 0.37, 0.17, 0.31}},
                                                     {{}, {},
                                                      {3.07, 0.85, 0.60, 0.40, 1.18},
                                                      {}, {}, {},
                                                      {3.45, 0.39, 0.47, 0.30, 0.48},
                                                      {3.09, 0.14, 0.18, 0.18, 0.37},
                                                      {},
                                                      {1.79, 3.61, 1.14, 0.62, 3.11},
                                                      {1.66, 3.59, 0.87, 0.46, 1.94},
                                                      {1.58, 2.68, 0.57, 0.34, 1.28},
                                                      {1.59, 1.97, 0.33, 0.25, 0.67},
                                                      {2.53, 0.74, 0.23, 0.17, 0.29}},
                                                     {{}, {}, {}, {}, {}, {}, {},
                                                      {4.53, 0.01, 0.08, 0.20, 0.90, 2.14, 0.25},
                                                      {},
                                                      {4.99, 3.53, 0.00, 0.65, 2.90, 8.19, 2.31},
                                                      {},
                                                      {3.10, 2.62, 0.16, 0.36, 1.41, 3.99, 0.46},
                                                      {2.75, 1.27, 0.05, 0.27, 2.07, 1.99, 0.82},
                                                      {3.24, 0.90, 0.13, 0.18, 0.32, 2.02, 0.00}},
                                                     {{}, {}, {}, {}, {}, {},
                                                      {6.57, 0.82, 0.0, 0.24, 0.82},
                                                      {5.09, 0.0, 0.0, 0.14, 0.89},
                                                      {},
                                                      {5.77, 6.34, 0.0, 0.62, 3.16},
                                                      {4.76, 5.00, 0.0, 0.48, 2.39},
                                                      {3.75, 3.60, 0.0, 0.34, 1.55},
                                                      {2.58, 2.42, 0.0, 0.26, 0.88},
                                                      {4.04, 0.26, 0.0, 0.16, 1.18}}};
        const bool short_sum = whole_short || p.k <= 256;
        const ShortCost *short_cost = short_costs[whole_short ? 1 : (triangular_c ? 2 : (p.beta != 0.f && p.m % 8 != 0 ? 3 : 0))];
        // The checked register-staged 256 x 256 tile beside them, in the same form (147 sizes of 640 to 7000 terms, 5 % rms), where 192 x 192 tiles
        // leave a nearly empty turn: (5416, 5112, 2456) 192 x 192 159 us, this 142, (3280, 3600, 2600) 86.2, 67.6; SYRK (4600, 2896) 128 x 128 88.2, this
        // 72.8.  Of 250 products of 900 to 8000 it takes 12, 0.93 of the time, one 2 % slower.
        constexpr int kStagedLargest = 3;
        static const RaggedCost staged_largest = {6.9, 0.98, 0.44, 0.0, 0.94, 1.10, 1.03, 0.08, 1.0, 1.0};
        const bool ragged_family = !f32 && !(whole64 && p.shape != MG_SHAPE_GENERAL && !triangular_c && p.k <= 192) && p.conv == nullptr && p.clip_m == 0 && p.clip_n == 0 &&
                                   dma_ragged_operands(p, alignment) && dma_offsets_fit(p, 192, 64);
        // FP16 operands that the direct-to-LDS kernels do not take (rows off 16 bytes, sizes that end inside a piece): the tiles whose pieces come from any
        // element (mfma_any_kernel.h), with 1, 2, 4 or 8 slices; for sums of up to 320 terms beside the checked register-staged ones, unsliced, which start
        // sooner and whose wavefronts write their parts of C one by one ((512, 1664, 128) 4.1 us on 64 x 64 of these, 5.2 of those, (1402, 6146, 64)
        // 11.9 us, 18.5 on 192 x 128; (143, 5204, 475) with beta 8.7, 7.5); up to 1024 beside the register-staged 256 x 256 tile ((4997, 5466, 896) 68 us, 79 on 256 x 128).
        // Their time in us: a fixed part; turns of one tile per compute unit and, per K-tile, what a turn, a busier chip, rows at odd elements (`odd`: the share
        // of a tile's rows) and operands along their rows take longer; the traffic of C (MB), of which rows off 16 bytes; and `more`: short sums a sum
        // that ends inside a K-tile and old columns of C that end inside a piece, per turn; long ones the second launch and the partial sums of slices.
        // Fitted to all tiles on 1700 sizes of 32 to 7000 and sums of 32 to 8192, a third each with odd and with padded leading dimensions (5 to 11 %,
        // register-staged 10 to 15 % rms).  Fitted to half and chosen for the other half: 1.018 times the fastest, 51 of 946 more than 5 % behind, up to 1.28.
        // Short sums on more than three 64 x 64 tiles per compute unit have costs of their own, with what the register-staged tiles' one-by-one ends take (rows and values of k
        // behind the last piece) and rounds of the work-groups that a compute unit holds: with those of all short sums, most of them on small grids, 27 % of 4700 such calls
        // were more than 5 % slower than on the best register-staged tile, up to 1.38 ((2816, 7337, 10) 28.3 / 36.0 us, (1137, 2758, 128) 9.2 / 10.7), with their own 12 %.
        struct AnyCost {
            double fixed, turn, busy, turn_ktile, busy_ktile, odd, lines, c, turn_beta, c_stray, more[2];
            double rows_behind, old_rows_behind, terms_behind, round, round_ktile;
        };
        static const TileChoice any_tiles[] = {{"hany16_256x128x64_w4x2", 256, 128, 64, 0.f, 0.f, 1},
                                               {"hany16_192x128x64_w2x4", 192, 128, 64, 0.f, 0.f, 1},
                                               {"hany16_128x128x64_w2x4", 128, 128, 64, 0.f, 0.f, 1},
                                               {"hany16_128x64x64_w4x2", 128, 64, 64, 0.f, 0.f, 1},
                                               {"hany16_64x64x64_w2x2", 64, 64, 64, 0.f, 0.f, 1},
                                               {"hmfma_64x64x64_w2x2", 64, 64, 64, 0.f, 0.f, 5},
                                               {"hmfma_128x64x64_w2x2", 128, 64, 64, 0.f, 0.f, 3},
                                               {"hmfma_128x128x64_w2x2", 128, 128, 64, 0.f, 0.f, 2},
                                               {"hmfma_256x256x64_w2x2", 256, 256, 64, 0.f, 0.f, 1}};
        constexpr int kAnyStaged = 5, kAnyCount = 9;         // index of the first register-staged one
        static const AnyCost any_costs[3][kAnyCount] = {{{3.96, 5.20, 0.0, 0.726, 0.0, 0.153, 0.192, 0.187, 0.685, 0.054, {0.0, 1.95}},
                                                         {3.52, 4.27, 1.82, 0.587, 0.0, 0.118, 0.201, 0.028, 0.129, 0.055, {0.0, 2.13}},
                                                         {2.87, 3.84, 0.0, 0.407, 0.0, 0.167, 0.153, 0.170, 0.359, 0.029, {0.0, 0.80}},
                                                         {4.07, 1.22, 0.55, 0.249, 0.0, 0.114, 0.117, 0.035, 0.132, 0.017, {0.0, 0.53}},
                                                         {4.38, 0.49, 0.45, 0.173, 0.0, 0.059, 0.043, 0.0, 0.121, 0.066, {0.0, 0.24}},
                                                         {4.84, 0.48, 0.0, 0.075, 0.118, 0.018, 0.040, 0.0, 0.102, 0.039, {0.12, 0.57}},
                                                         {6.01, 0.70, 0.0, 0.137, 0.167, 0.034, 0.102, 0.0, 0.067, 0.058, {0.19, 1.70}},
                                                         {7.04, 1.36, 0.0, 0.400, 0.069, 0.0, 0.041, 0.0, 0.283, 0.105, {0.34, 4.13}},
                                                         {5.77, 7.98, 0.0, 0.803, 0.786, 0.172, 0.419, 0.0, 1.017, 0.087, {0.0, 11.2}}},
                                                        {{5.26, 4.19, 0.0, 0.678, 0.113, 0.150, 0.0, 0.264, 1.347, 0.024, {1.09, 0.337}},
                                                         {4.65, 3.33, 0.0, 0.571, 0.070, 0.115, 0.003, 0.294, 1.058, 0.009, {1.35, 0.359}},
                                                         {3.27, 3.55, 0.0, 0.435, 0.066, 0.100, 0.012, 0.215, 0.807, 0.040, {1.72, 0.365}},
                                                         {4.57, 0.53, 0.0, 0.331, 0.015, 0.077, 0.008, 0.271, 0.423, 0.045, {1.89, 0.462}},
                                                         {4.63, 0.0, 0.40, 0.256, 0.002, 0.033, 0.025, 0.048, 0.294, 0.141, {1.79, 0.419}},
                                                         {}, {}, {},
                                                         {5.65, 7.07, 4.47, 1.103, 0.127, 0.144, 0.028, 0.0, 5.391, 0.128, {0.0, 0.0}}},
                                                        {{4.84, 5.96, 0.0, 0.584, 0.0928, 0.165, 0.176, 0.114, 1.45, 0.0513, {0.0, 0.473}},
                                                         {4.54, 4.67, 0.0, 0.518, 0.0, 0.127, 0.168, 0.129, 1.32, 0.0479, {0.0667, 0.479}},
                                                         {4.08, 4.01, 0.0, 0.411, 0.0, 0.141, 0.144, 0.125, 0.86, 0.0254, {0.0, 0.0855}},
                                                         {4.53, 1.87, 0.0, 0.259, 0.0, 0.0965, 0.0514, 0.0479, 0.311, 0.0217, {0.0, 0.0689}},
                                                         {5.82, 0.233, 0.0, 0.166, 0.0, 0.0618, 0.0264, 0.398, 0.194, 0.0261, {0.00326, 0.0385}},
                                                         {5.84, 0.0, 0.0, 0.115, 0.0934, 0.0216, 0.0, 0.3, 0.187, 0.00816, {0.0424, 0.0}, 0.0649, 0.364, 0.221, 0.0945, 0.0278},
                                                         {5.62, 0.0, 0.0, 0.0857, 0.145, 0.0428, 0.0, 0.125, 0.438, 0.0208, {0.0, 0.0768}, 0.27, 0.959, 0.401, 1.92, 0.29},
                                                         {6.54, 0.0, 0.0, 0.0, 0.212, 0.0553, 0.0, 0.105, 1.12, 0.0388, {0.0, 0.365}, 0.645, 2.56, 0.609, 2.72, 0.527},
                                                         {8.64, 2.09, 0.0, 0.647, 0.78, 0.12, 0.0694, 0.0997, 3.56, 0.053, {0.0, 2.68}, 3.57, 9.17, 1.15, 1.2, 0.599}}};
        // (long sums of a triangle of C, on the largest of them: fitted to half of 300 SYRK of 2000 to 7000 rows and 321 to 6000 terms; see `uneven` below)
        static const AnyCost triangle_largest = {8.3, 8.2, 0.0, 1.03, 0.45, 0.076, 0.009, 0.22, 0.0, 0.0, {0.0, 0.0}};
        const bool any_short = p.k <= 320;
        const bool any_family = !f32 && p.conv == nullptr && p.clip_m == 0 && p.clip_n == 0 && p.k >= 8 && !dma_ragged_operands(p, alignment);
        // The register-staged FP16 kernels transpose operands that are not contiguous along k on their way to
        // LDS; the smaller the tile, the more that shows.  Measured rates relative to the (m, k) order (A along m,
        // B along k; tiles up to 128 x 64 / up to 256 x 128 / 256 x 256): both operands along k 1.10 / 1.06 / 1.02,
        // A along m and B along n 0.93 / 0.97 / 0.98.
        auto staged_f16 = [&](const TileChoice &t) {
            const int cls = t.bm * t.bn <= 128 * 64 ? 0 : (t.bm * t.bn <= 256 * 128 ? 1 : 2);
            static const double both_k[3] = {1.10, 1.06, 1.02}, neither_k[3] = {0.93, 0.97, 0.98};
            if (p.a_trans && !p.b_trans) return both_k[cls];
            if (!p.a_trans && p.b_trans) return neither_k[cls];
            return 1.0;
        };
        // FP32: a single work-group keeps the MFMA pipes of its compute unit nearly busy, so work-groups that share
        // a compute unit take turns rather than overlap (128 x 128 at k = 2048: 256 / 288 / 512 / 768 / 1024 tiles
        // take 128 / 233 / 249 / 368 / 474 us): rounds of 256 tiles whatever the tile, at a rate that rises from
        // `per_group` (one round) towards `ceiling` (many), plus what a round of small tiles costs on top
        // (0 / 0 / 1 / 2 / 1.8 us from the largest tile to the smallest: first loads and the epilogue).
        // The two tiles of which a compute unit holds a single work-group run with eight wavefronts (two per SIMD:
        // one hides the other's barrier and LDS waits; 4096^3 in the steady power state 1036 -> 932 us for 256 x 256,
        // 973 -> 950 us for 256 x 128; the four-wavefront variants stay in the table).
        // Rates: turns * tile flops / time of every tile on the squares 1024^3 to 6144^3 (the four operand orders run
        // alike since the operands along m / n keep their memory layout in LDS): one turn gives `per_group`, many
        // turns `ceiling`.
        static const TileChoice f32_tiles[] = {{"smfma_256x256x32_w2x4", 256, 256, 32, 0.591f, 0.591f, 1},
                                               {"smfma_256x128x32_w4x2", 256, 128, 32, 0.587f, 0.583f, 1},
                                               {"smfma_128x128x32_w2x2", 128, 128, 32, 0.588f, 0.566f, 2},
                                               {"smfma_128x64x32_w2x2", 128, 64, 32, 0.582f, 0.54f, 3},
                                               {"smfma_64x64x32_w2x2", 64, 64, 32, 0.571f, 0.565f, 5},
                                               {"ssplit_256x128x32_w4x2", 256, 128, 32, 0.f, 0.f, 1},
                                               {"ssplit_128x128x32_w2x4", 128, 128, 32, 0.f, 0.f, 1}};
        constexpr int kSplit = 5;           // index of the first kernel on the bf16 matrix pipes
        // Their time in us: turns of one tile per compute unit, each a fixed part and, per K-tile of 32, a part that grows with the square of
        // the share of the chip that is busy (the power limit); and the traffic of C per MB.  Fitted to both tiles with 1 to 8 slices on 13
        // sizes in two orders, one turn and several: 256 x 128 tiles take 2.0 us per K-tile on up to 128 compute units, 2.5 on 224, 2.7 on
        // all (512^3 40.2 us, 1000^3 73.0, 2048^3 141, (1673, 4032, 554) 57, (8192, 1024, 512) 56, 4096^3 735); 128 x 128 tiles 1.07 on
        // 64, 1.12 on 144, 1.35 on three turns of 192, 1.48 on all (512^3 23.5, 1000^3 40.8, 1500^3 60, 3000^3 405, 2048^3 104, 4096^3 788).
        // These are for both operands along k; an operand along its rows takes two transposing reads per fragment (128 x 128 tiles,
        // kk / mk / mn / kn: (4096, 256, 4096) 149 / 162 / 164 / 158, (3072, 3072, 1536) 217 / 227 / 227 / 223; 256 x 128 250 / 252 / 258 / 253)
        struct SplitCost {
            double turn, ktile, ktile_load, c_mb;
        };
        static const SplitCost split_costs[2] = {{8.2, 1.95, 0.75, 0.18}, {5.8, 1.06, 0.41, 0.16}};
        static const double f32_round_cost[5] = {0.0, 0.0, 1.0e6, 2.0e6, 1.8e6};
        const TileChoice *tiles = f32 ? f32_tiles : (any_family ? any_tiles : f16_tiles);
        const int count = f32 ? 7 : (any_family ? kAnyCount : (ragged_family ? 14 : 9));
        const int smallest = f32 ? 4 : (any_family ? -1 : (ragged_family ? kRaggedSmallest : 7));
        bool tried[14] = {false};
        // work-groups that do something: of a product whose C is a triangle, the tiles that touch it (as the kernels skip the others)
        const bool triangle = p.shape == MG_SHAPE_C_LOWER || p.shape == MG_SHAPE_C_UPPER;
        // a triangular operand: tiles with sums of every length up to k, on average half (FP32; see the end of the ranking for FP16)
        const bool narrowed = p.shape != MG_SHAPE_GENERAL && !triangle;
        auto wanted_tiles = [&](int bm, int bn) {
            const int64_t across_m = ceil_div(tm, bm), across_n = ceil_div(tn, bn);
            return triangle ? triangle_tiles(p.shape == MG_SHAPE_C_LOWER, across_m, across_n, bm, bn) : across_m * across_n;
        };
        // estimated time (in 1e-6 us) of tile i with the sum cut into `slices`
        const bool any_large = any_family && any_short && wanted_tiles(64, 64) > 3 * kComputeUnits;
        auto estimate = [&](int i, int slices) {
            const int64_t blocks = wanted_tiles(tiles[i].bm, tiles[i].bn) * slices;
            if (any_family) {
                const AnyCost &cost = triangle && !any_short && i == kAnyCount - 1 ? triangle_largest : any_costs[any_short ? (any_large ? 2 : 0) : 1][i];
                // (the checked tiles of a triangle have a work-group for each tile of the square, which go to the 32 groups of eight compute units in turn, and the busiest group has
                // a tenth more wanted ones than its share: 8 of 210 on 20 x 20 tiles and of the lower 231 on 21 x 21, 9 of the upper ones and of 253 on 22 x 22, which take a
                // second turn.  SYRK on 256 x 256, (5283, 274) lower 28.2 us, (5287, 480) upper 45.2, (5120, 140) 24.4, (5435, 100) 34.7, 23.8 on 128 x 128; two of these at once
                // on a compute unit, (3640, 207) 17.2 on 29 x 29, (3865, 220) 24.1 on 31 x 31, 17.7 on the direct-to-LDS ones)
                const bool uneven = triangle && i >= kAnyStaged && (any_large || !any_short);
                const double x = static_cast<double>(blocks) / kComputeUnits, filled = uneven ? (p.shape == MG_SHAPE_C_UPPER ? 1.11 : 1.105) * x : x, turns = ceil(filled), ktiles = static_cast<double>(ceil_div(ceil_div(p.k, 64), slices));
                const double bm = tiles[i].bm, bn = tiles[i].bn;
                const double odd = ((p.lda % 2 != 0 ? bm : 0.0) + (p.ldb % 2 != 0 ? bn : 0.0)) / (bm + bn), lines = ((p.a_trans ? 0.0 : bm) + (p.b_trans ? bn : 0.0)) / (bm + bn);
                const double c_mb = 2.0e-6 * static_cast<double>(p.m) * static_cast<double>(p.n) * (triangle ? 0.5 : 1.0);
                double us = cost.fixed + turns * cost.turn + x * cost.busy + ktiles * (turns * (cost.turn_ktile + cost.lines * lines) + x * cost.busy_ktile + (turns + x) * cost.odd * odd);
                us += cost.c * c_mb + (p.beta != 0.f ? turns * cost.turn_beta : 0.0);
                if (slices == 1 && p.ldc % 8 != 0) us += cost.c_stray * c_mb;
                if (any_short) us += turns * ((p.k % 64 != 0 ? cost.more[0] : 0.0) + (p.beta != 0.f && p.m % 8 != 0 ? cost.more[1] : 0.0));
                if (any_short && any_large) {
                    const double rounds = ceil(filled / tiles[i].resident), rows = uneven ? 0.0 : static_cast<double>(p.m % 8) / 8.0;
                    us += turns * (rows * (cost.rows_behind + (p.beta != 0.f ? cost.old_rows_behind : 0.0)) + cost.terms_behind * static_cast<double>(p.k % 8) / 8.0);
                    us += rounds * (cost.round + cost.round_ktile * ktiles);
                }
                if (!any_short && slices > 1) us += cost.more[0] * (1.0 + 0.1 * slices) + cost.more[1] * 2.0 * slices * c_mb;
                // (a nearly full turn of 64 x 64 tiles and long sums runs 5 to 8 % above that: (1672, 560, 3264) 22.9 us, 128 x 64 in two slices 22.3)
                if (!any_short && i == kAnyStaged - 1 && slices == 1 && x > 0.5 && x <= 1.0 && ktiles >= 30.0) us *= 1.07;
                // (masked stores of a triangle fetch the old C piece by piece there: SYRK 690 x 1408 with beta 13.9 us on 64 x 64 register-staged tiles, 10.7 on these)
                // (many tiles: masked ends go one by one at any height of C, and those of the diagonal are waited for once.  With this and the turns above 276 SYRK of up to 320
                // terms, not those it was fitted to, take 1.012 times the fastest of the square tiles, at most 1.18; with a charge per turn 1.033, at most 1.84: (5409, 103) with
                // beta 63.1 us, 34.2 on 128 x 128.  161 of more terms 1.010, with that charge and no 256 x 256 tiles beyond 1024 terms 1.056: (5551, 587) with beta 88.5 on these,
                // 57.1 on 128 x 128, (5077, 3771) 116 on these, 181)
                if (uneven) {
                    const bool old = p.beta != 0.f;
                    if (!any_short) us += old ? 18.9 : 0.0;
                    else if (bm > 128.0) us += old ? 14.0 : 2.5;
                    else if (bm > 64.0) us += old ? 8.8 : 0.9;
                    else us += old ? 4.3 : 0.6;
                    if (any_short && p.a_trans) us += x * (bm > 128.0 ? (old ? 2.8 : 0.74) : bm > 64.0 ? (old ? 1.4 : 0.7) : (old ? 0.32 : 0.08));
                } else if (i >= kAnyStaged && triangle) us += turns * (p.beta != 0.f ? 2.5 : 0.4);
                return us * 1.0e6;
            }
            const double tile_flops = 2.0 * tiles[i].bm * tiles[i].bn * static_cast<double>(p.k) / slices;
            const int64_t full = static_cast<int64_t>(kComputeUnits) * tiles[i].resident;   // work-groups the chip holds
            double order = 1.0;
            if (!f32 && tiles[i].tag[1] == 'm') order = staged_f16(tiles[i]);
            // sliced sums run the large register-staged tiles about a tenth below their rate (256 x 8192 x 8192 with
            // both operands along k in four slices: 53-55 us against 48 us on the direct-to-LDS tile of that size)
            if (!f32 && tiles[i].tag[1] == 'm' && slices > 1 && tiles[i].bm * tiles[i].bn >= 256 * 128) order *= 0.9;
            if (!f32 && i == kDeep && !(p.a_trans && !p.b_trans)) order = 0.95;
            // the 128 x 128 direct-to-LDS tile is slower with A along k (3.7-3.8 against 4.0)
            if (!f32 && i == 2 && p.a_trans) order = 0.94;
            // ragged FP16 problems run the bounds-checked flavour (FP32: see below)
            const bool ragged = tm % tiles[i].bm || tn % tiles[i].bn || p.k % tiles[i].bk || tm != p.m || tn != p.n;
            // (rates against the whole-tile flavour, one work-group per compute unit / more, and what the larger tiles' checked ends
            // cost on top, fitted to every bounds-checked tile with 1 to 14 slices on 13 sizes in three orders, odd rows: (1672, 561,
            // 3265) 31.9 us on 256 x 256 in 8 slices, 22.9 on 128 x 64 in 4; (295, 7412, 1245) 128 x 128 34.7, 64 x 64 25.4; (4379, 256,
            // 4608) 256 x 256 in 8 40.7, 128 x 128 in 4 35.8; (2881, 3483, 37) 26.0, 17.3; (448, 609, 2741) 128 x 128 in 8
            // 17.9, 64 x 64 in 4 14.2; (8201, 1031, 2051) 256 x 256 64, 128 x 128 91)
            double ends = 0.0;
            if (!f32 && ragged) {
                const int area = tiles[i].bm * tiles[i].bn;
                const bool several = blocks > kComputeUnits;
                if (area >= 256 * 256) { order *= 0.9; ends = 4.0e6; }
                else if (area >= 256 * 128) { order *= 0.77; ends = 8.0e6; }
                else if (area >= 128 * 128) { order *= several ? (slices > 1 ? 0.95 : 0.8) : 0.75; ends = 2.0e6; }
                else if (area >= 128 * 64) { order *= several ? (slices > 1 ? 0.85 : 0.7) : 0.7; ends = 1.0e6; }
                else { order *= several ? 0.85 : 0.65; ends = 1.0e6; }
            }
            // rate of a compute unit that holds u work-groups at once: ceiling * (1 - (1 - per_group / ceiling)^u)
            // (measured on the 64 x 64 FP16 tile: 1.33 / 1.85 / 2.02 / 2.11 for u = 1..4, the formula gives
            // 1.31 / 1.86 / 2.09 / 2.18)
            auto shared_rate = [&](int64_t u) {
                const double idle = 1.0 - (tiles[i].per_group < tiles[i].ceiling ? tiles[i].per_group / tiles[i].ceiling : 1.0);
                return tiles[i].ceiling * (1.0 - pow(idle, static_cast<double>(u)));
            };
            double time;
            if (ragged_family && short_sum) {
                const ShortCost &cost = short_cost[i];
                const double x = static_cast<double>(blocks) / kComputeUnits, ktiles = static_cast<double>(ceil_div(p.k, 64)) * (p.b_trans ? 1.12 : 1.0);
                const double updates = p.beta != 0.f ? cost.fixed_beta + ceil(x) * cost.turn_beta + x * cost.busy_beta : 0.0;
                return 1.0e6 * (cost.fixed + ceil(x) * (cost.turn + cost.ktile * ktiles) + x * cost.busy + updates);
            }
            const bool large_staged = ragged_family && i == kStagedLargest;
            if (!f32 && (i >= kRagged || large_staged)) {
                const RaggedCost &cost = large_staged ? staged_largest : ragged_costs[i - kRagged];
                double each = p.a_trans ? (p.b_trans ? 1.0 : cost.both_k) : (p.b_trans ? cost.neither_k : cost.one_k);
                if (p.a_trans && p.lda % 64) each *= 1.0 + cost.stray_rows;
                else if (!p.b_trans && p.ldb % 64) each *= 1.0 + 0.5 * cost.stray_rows;
                const double ktiles = static_cast<double>(ceil_div(ceil_div(p.k, 64), slices)) * each;
                auto turn = [&](double load) {
                    return load <= 1.0 ? cost.turn + ktiles * (cost.ktile + cost.ktile_load * load * load)
                                       : cost.turn + ktiles * (cost.ktile + cost.ktile_load + cost.second);
                };
                const int64_t whole = blocks / full, rest = blocks % full;
                double us = (large_staged ? 3.4 : 0.5) + static_cast<double>(whole) * turn(tiles[i].resident) +
                            (rest > 0 ? turn(static_cast<double>(rest) / kComputeUnits) : 0.0);
                us += cost.c * 2.0 * static_cast<double>(p.m) * static_cast<double>(p.n) * (p.beta != 0.f ? 2.0 : 1.0) * (triangle ? 0.5 : 1.0) / 4.5e6;
                // (the masked stores of a triangle, which fetch the old C tile by tile: what a turn takes longer than on 64 x 64 tiles, without / with
                // beta, 105 SYRK of 64 to 2800; (2824, 256) with beta 22.3 us on 192 x 192 tiles, 13.6 on 64 x 64, (72, 64) 5.6 on 128 x 128, 4.1)
                static const double masked[2][5] = {{2.6, 1.5, 0.9, 0.3, 0.0}, {8.7, 5.0, 3.1, 0.3, 0.0}};
                if (triangle && slices == 1 && !large_staged) us += masked[p.beta != 0.f][i - kRagged] * static_cast<double>(whole + (rest > 0 ? 1 : 0));
                if (triangle && large_staged) us *= 1.1;
                // (few tiles: a K-tile is a load's latency; (72, 2224) 13.2 us unsliced, 9.0 in slices)
                if (triangle && blocks <= kComputeUnits / 4) us += 0.1 * ktiles;
                if (slices > 1)
                    us += 3.0 + 0.2 * slices + cost.sums * (4.0 * slices + 6.0) * static_cast<double>(p.m) * static_cast<double>(p.n) * (triangle ? 0.5 : 1.0) / 4.0e6;
                return us * 1.0e6;
            }
            if (f32 && i >= kSplit) {
                const SplitCost &cost = split_costs[i - kSplit];
                const double ktiles = static_cast<double>(ceil_div(ceil_div(p.k, tiles[i].bk), slices)) * (p.a_trans && !p.b_trans ? 1.0 : 1.05);
                auto turn = [&](double load) { return cost.turn + ktiles * (cost.ktile + cost.ktile_load * load * load); };
                // (a triangle's tiles: those of the shader engine that gets most.  SYRK, us, while all counted as equal / now: (3840, 458) 100 / 76,
                // (2660, 1088) upper 101 / 73, (3728, 2310) 338 / 294, (5520, 576) 193 / 169; 3 us of host time at the most)
                int64_t share = blocks;
                if (triangle && blocks <= (slices == 1 ? 4 : 2) * kComputeUnits)
                    share = busiest_engine_tiles(p.shape == MG_SHAPE_C_LOWER, ceil_div(tm, tiles[i].bm), ceil_div(tn, tiles[i].bn), tiles[i].bm, tiles[i].bn, slices);
                const double turns = static_cast<double>(share) / kComputeUnits;
                double us;
                if (narrowed) {
                    // (sums of half the length on average, the longest first; TRMM 3000 on 128 x 128 tiles 208 us, 4096 421, 8192 2970)
                    us = turns > 1.0 ? std::max(1.0, 0.5 * turns + 0.2) * turn(1.0) : turn(turns);
                } else {
                    us = floor(turns) * turn(1.0) + (turns > floor(turns) ? turn(turns - floor(turns)) : 0.0);
                }
                time = 1.0e6 * (us + cost.c_mb * 4.0e-6 * static_cast<double>(p.m) * static_cast<double>(p.n) * (p.beta != 0.f ? 2.0 : 1.0));
                // (nothing that the FP32 pipes do as fast: the estimates are within about 7 % of each other's truth.  us, FP32 pipes /
                // bf16 pipes at estimates less than that apart: (2656, 3207, 1150) 167 / 184, (560, 1920, 3746) 82 / 86, (5602, 5340, 266) 159 /
                // 157, (280, 4504, 3032) 78 / 77.  A triangle's tiles win at such estimates: SYRK 2048 118 / 86, 4096 554 / 499, 2194 x 2873 180 / 128)
                if (p.shape == MG_SHAPE_GENERAL) time *= 1.07;
            } else if (f32) {
                // work-groups take turns on a compute unit: ceil(blocks / 256) turns of one tile each, whether the
                // compute units hold them all at once or are refilled as work-groups retire (squares of 1024 to 6144
                // on every tile: within 6 % of this, the small tiles a little better where the last turn is thin)
                double rounds = static_cast<double>(ceil_div(blocks, kComputeUnits));
                if (narrowed && rounds > 1.0) rounds = std::max(1.0, 0.55 * static_cast<double>(blocks) / kComputeUnits);
                const double up = ceil(rounds);
                // (the bounds-checked flavour runs its whole K-tiles on the fast flavour's schedule and the end of the sum on
                // checked loads: 0.75 of these rates for a single turn, which has no other work-group's arithmetic to hide
                // the checked part behind, 0.85 for two or more work-groups per compute unit; and every further work-group
                // of a compute unit adds half a turn's fixed cost.  From 64 x 64 tiles, us measured / this estimate:
                // (1000, 1001, 999) unsplit 21.5 / 21.1, two slices 27.0 / 26.7; (4097, 129, 4095) less its fringe unsplit
                // 71 / 81, two slices 46.7 / 47.5, four 46.2 / 44.7, eight 54.9 / 48.4; (1025, 1030, 1000) less its fringe
                // row unsplit 36.3 / 36.6, two slices 35.2 / 37.1, four 38.1 / 36.8)
                const double rate = (tiles[i].ceiling - (tiles[i].ceiling - tiles[i].per_group) / up) * (ragged ? (up <= 1.0 ? 0.75 : 0.85) : 1.0);
                // (work-groups that are resident together pay the fixed cost of a turn once)
                time = rounds * tile_flops / rate + (blocks <= full ? (ragged ? 1.0 + 0.5 * (rounds - 1.0) : 1.0) : rounds) * f32_round_cost[i];
            } else if (blocks < full) {
                // the chip is not full: ceil(blocks / 256) work-groups share a compute unit
                const int64_t per_unit = ceil_div(blocks, kComputeUnits);
                double rate = shared_rate(per_unit);
                // FP16 runs against the power limit: when some compute units hold fewer work-groups than the
                // busiest ones (or none), the busy ones clock higher.  With `load` = the chip's summed rate as a
                // fraction of the rate with every compute unit as busy as the busiest, the gain is load^-e, at
                // most 1.4; e fitted per kernel: 256 x 256 direct-to-LDS 0.55 (144 tiles at 3072^3 run at 6.7
                // Mflop/us per compute unit against 4.8 on a full chip), 256 x 128 0.3 (direct-to-LDS and
                // register-staged), 128 x 128 direct-to-LDS 1.3 when the busiest compute units hold two work-groups
                // (324 tiles at 2304^3: 4.8 Mflop/us against 3.6) but 0.1 with one, its four-stage sibling 0.4, the smaller register-staged
                // kernels 0.1; the bounds-checked flavour shows no gain; the 128 x 128 direct-to-LDS tile at most 1.2
                if (!ragged || i == 3) {
                    const int64_t busiest = blocks - static_cast<int64_t>(kComputeUnits) * (per_unit - 1);
                    const double lower = per_unit > 1 ? shared_rate(per_unit - 1) : 0.0;
                    const double load = (static_cast<double>(busiest) * rate + static_cast<double>(kComputeUnits - busiest) * lower) /
                                        (static_cast<double>(kComputeUnits) * rate);
                    const double exponent = i == 0 ? 0.55 : (i == 1 ? 0.5 : (i == kDeep ? 0.4 : (i == 2 ? (per_unit > 1 ? 1.3 : 0.1) : (tiles[i].bm == 256 ? 0.3 : 0.1))));
                    const double boost = pow(load, -exponent);
                    const double most = i == 2 ? 1.2 : 1.4;
                    rate *= boost < most ? boost : most;
                }
                time = static_cast<double>(per_unit) * tile_flops / (rate * order);
            } else {
                // whole rounds of `full` work-groups at the ceiling, then the rest.  One work-group per compute
                // unit quantises sharply (576 tiles take three rounds).  FP16 kernels with several resident
                // work-groups: the rest is a round of its own with u = ceil(rest / 256) work-groups per compute
                // unit at their shared rate, four fifths of it exposed (it starts while the round before drains);
                // measured at k = 2048, 512 / 768 / 1024 / 1280 tiles: 128 x 128 direct-to-LDS 37 / 59 / 70 / 91 us
                // (this model: 34 / 57 / 68 / 91), register-staged 41 / 61 / 83 / 104 (38 / 58 / 76 / 96).  The
                // fastest FP16 kernel is an exception of its own: its partial last round runs on fewer compute
                // units at a higher clock (400 tiles take 1.7 rounds' time, 576 tiles 2.5)
                const double x = static_cast<double>(blocks) / static_cast<double>(full);
                const double whole = floor(x);
                const double round_time = tiles[i].resident * tile_flops / (tiles[i].ceiling * order);
                if (x == whole) time = x * round_time;
                else if (i == 0) time = (x + 0.25) * round_time;
                else if (tiles[i].resident == 1) time = (whole + 1.0) * round_time;
                else {
                    const int64_t rest = blocks - static_cast<int64_t>(whole) * full;
                    const int64_t u = ceil_div(rest, kComputeUnits);
                    time = whole * round_time + 0.8 * static_cast<double>(u) * tile_flops / (shared_rate(u) * order);
                }
            }
            // the kernels with three and four stages: their first loads and the epilogue beside the loop's rate (128 x 128 tiles:
            // 24 K-tiles on 144 compute units 14.7 us, 64 on 128 units 26.8 us, 16 on 64 units 10.7 us)
            if (!f32 && (i == 1 || i == kDeep)) time += 2.0e6;
            time += ends;
            // split-K: the partial sums are written and read back (8 bytes per slice and output at ~4 TB/s) by
            // a second launch (2.5 us; 4 us behind the bounds-checked FP32 flavour, fitted with the rates above)
            // (FP32: half of that traffic where only a triangle is written; SYRK 4096 on 256 x 128 tiles in 4 slices 494 us, 641 unsliced, 555 on
            // the FP32 pipes)
            const double sums = (4.0 * slices + 8.0) * static_cast<double>(p.m) * static_cast<double>(p.n) * (f32 && triangle ? 0.5 : 1.0);
            if (slices > 1) time += 1.0e6 * ((f32 && i >= kSplit ? 6.0 : (f32 && ragged ? 4.0 : 2.5)) + sums / 4.0e6);
            // (what a call takes beside its turns, in the constants of the others: 512^3 on 64 x 64 tiles 10.9 us, 9.1 without, 1024^3 19.7, 16.5)
            if (f32 && i < kSplit) time += 1.0e6;
            return time;
        };
        // each tile's estimate with the slices that suit it and the workspace, ranked once for all attempts
        struct Ranked {
            int slices;                      // 0: not a candidate
            double time;
        } ranked[14] = {};
        const bool in_place = p.clip_m != 0 || p.clip_n != 0;
        for (int i = 0; i < count; ++i) {
            // (short sums are the traffic of C, which the small tiles overlap better: (3870, 5248, 64) 45.7 / 40.0 us on the 64 x 64 tile of the
            // FP32 pipes, (2303, 2721, 64) 18.1 / 17.7, (6000, 700, 129) 20.7 / 21.5, (4096, 4096, 256) 63.4 / 73.4)
            if (f32 && i >= kSplit && (p.k < 128 || p.fp32_pipes)) continue;
            // FP32 work-groups take turns on a compute unit, so unequal tiles (skipped ones, narrowed K ranges) only pay off where a compute
            // unit gets many of them: of the kernels on the FP32 pipes the smallest (SYRK 4096: 974 / 923 / 695 / 618 us from the 256 x 256
            // to the 64 x 64 tile, TRMM 950 / 614 / 596 / 541).  Those on the bf16 pipes are ranked beside it (us, unsliced, FP32 pipes 64 x 64 /
            // bf16 pipes 256 x 128 / 128 x 128: SYRK 1146 x 1056 39 / 82 / 51, 2048 120 / 147 / 86, 3072 255 / 223 / 268, 4096 555 / 641 / 558,
            // 8192 4140 (128 x 64: 4102) / 3620 / 3757; TRMM 1000 31 / 82 / 53, 3000 241 / 239 / 208, 4096 527 / 450 / 421, 8192 3914 / 2741 / 2970)
            if (f32 && p.shape != MG_SHAPE_GENERAL && i < kSplit - 1) continue;
            if (in_place && i > 2 && i != kDeep) continue;           // (no other tile has the flavour, and it is not sliced)
            // FP32 with a short K is bound by the traffic of C, which the large tiles overlap worst (one epilogue per
            // compute unit at a time).  us, the tile the estimate would take (256 x 256 or 128 x 128) / 128 x 64 / 64 x 64,
            // beta != 0: (8192, 8192, 64) 200 / 154 / 157, (8192, 8192, 256) 351 / 310 / 322, (8192, 8192, 512) 574 / 534 / 551,
            // (4096, 4096, 160) 60 / 59 / 54, (3000, 3000, 256) 67 / 53 / 47, (2048, 2048, 512) 41 / 40 / 36, (5000, 5000,
            // 64) - / 69 / 70; beta = 0: (2048, 2048, 160) 18.1 / 17.4 / 16.7, (3000, 3000, 160) 43 / 38 / 33, from
            // k = 256 on within 2 %; ragged problems of several turns whose 128 x 64 tiles need no more of them stay
            // on those: (1393, 4318, 136) 31.3 / 33.9 (five turns against nine: (3000, 3000, 160) above)
            if (f32 && i < kSplit && p.k <= 128 && tiles[i].bm * tiles[i].bn > 128 * 64) continue;
            if (f32 && i < kSplit && p.shape == MG_SHAPE_GENERAL && p.k <= (p.beta != 0.f ? 512 : 192)) {
                const int64_t turns64 = ceil_div(ceil_div(tm, 64) * ceil_div(tn, 64), kComputeUnits);
                const int64_t turns128 = ceil_div(ceil_div(tm, 128) * ceil_div(tn, 64), kComputeUnits);
                const bool whole = tm % 128 == 0 && tn % 64 == 0 && p.k % 32 == 0;
                const bool wide = whole ? p.m * p.n > 25000000 : p.k > 128 && turns64 >= 6 && 2 * turns128 <= turns64;
                if (tiles[i].bm * tiles[i].bn > (wide ? 128 * 64 : 64 * 64)) continue;
            }
            if (ragged_family && short_sum) {
                // (the whole tiles' costs are for tiles that divide C)
                if (short_cost[i].fixed == 0.0 || (i < kRagged && whole_short && (p.m % tiles[i].bm != 0 || p.n % tiles[i].bn != 0))) continue;
            } else if (ragged_family && i > 3 && i < kDeep) {
                continue;            // (beside these the smaller register-staged kernels have nothing to gain from longer sums)
            }
            // (a single turn of two stages and a few K-tiles: (7936, 256, 320) 6.8 us, 5.8 on other tiles)
            if (ragged_family && !short_sum && i == 2 && p.k <= 512 && wanted_tiles(128, 128) <= kComputeUnits) continue;
            // (the checked 256 x 256 tile only where there is no whole one and all its sums are as long; for triangles of C if no masked stores fetch
            // the old C, SYRK (5344, 2384) with beta 147 us, 88 on 192 x 192, and few tiles, whose grid holds the others too: (5512, 4032), 253 of 484,
            // 175 us, 114)
            if (ragged_family && i == kStagedLargest && (narrowed || (triangle && (p.beta != 0.f || wanted_tiles(256, 256) > kComputeUnits * 3 / 4)) || (p.m % 256 == 0 && p.n % 256 == 0 && p.k % 64 == 0))) continue;
            // (tiles of a triangle are counted for heights that are multiples of the width)
            if (!f32 && triangle && (any_family || i >= kRagged) && tiles[i].bm % tiles[i].bn != 0) continue;
            // (and only square tiles have a grid of the wanted ones: SYRK (3603, 578) 256 x 128 37.9 us, 128 x 128 register-staged 25.2)
            if (any_family && triangle && tiles[i].bm != tiles[i].bn) continue;
            if (any_family && !any_short && (any_costs[1][i].fixed == 0.0 || (i == kAnyCount - 1 && !triangle && p.k > 1024))) continue;
            // (of fewer than eight rows or columns, which no other tile takes, the largest one only in grids that nearly fill the chip, of both operands along k or of a long op(A)
            // with op(B) along k: (60393, 7, 401), both along k, 19.4 us, 32.0 on the shared-sum kernel below, (49555, 3, 540) 22.9 / 35.5; else (7, 9000, 700) 54.7 / 12.2, both
            // along k 25.0 / 9.8, (39488, 4, 464) 22.4 / 17.6, (7, 60462, 747) 89 / 52)
            if (any_family && !any_short && (p.m < 8 || p.n < 8) && !(!p.b_trans && (p.a_trans || p.m > p.n) && wanted_tiles(256, 256) > 160)) continue;
            const bool last = i == smallest;
            const int64_t ktiles = ceil_div(p.k, tiles[i].bk);
            const int64_t blocks = wanted_tiles(tiles[i].bm, tiles[i].bn);
            // slices tried: none; for the smallest tile the factor of the sweep's rule; for grids that do not
            // fill the chip powers of two that leave every slice at least four K-tiles
            int options[6] = {1, 0, 0, 0, 0, 0};
            int n_options = 1;
            // (a triangular operand already leaves half of the work-groups short sums: slices only where tiles are few; TRMM FP16 3968 x 1181
            // 55 us unsliced, 76 in two slices, 1797 x 221 73 / 37)
            // (FP16 triangles of C below 10 us: what slices gain the second launch takes; unsliced / in 4 slices, us on the device | calls in a
            // row: 200 x 1000 T 7.5 / 8.2 | 8.3 / 10.9, 256 x 2048 T 9.7 / 8.4 | 9.7 / 10.0, 256 x 4096 T 15.9 / 9.8 | 15.9 / 10.3)
            const double unsliced = estimate(i, 1);
            const bool short_triangle = !f32 && triangle && unsliced < (i >= kRagged ? 5.0e6 : 10.0e6);
            if (!in_place && !short_triangle && !(narrowed && blocks > kComputeUnits / 4)) {
                if (last && !ragged_family) options[n_options++] = pick_split(blocks, ktiles);
                if (blocks < 2 * kComputeUnits && (any_family ? i < kAnyStaged : !ragged_family || i >= kRagged))
                    for (int sl = 2; sl <= (ragged_family || any_family ? 8 : 16) && ktiles / sl >= 4; sl *= 2) options[n_options++] = sl;
            }
            for (int o = 0; o < n_options; ++o) {
                const int sl = options[o];
                if (sl < 1 || (o > 0 && sl == 1)) continue;
                // (a fringe work-group takes a compute unit of its own beside these kernels' tiles: only behind two turns of tiles and more;
                // (513, 515, 2000) 19.4 / 24.7 us, (4097, 129, 4095) 51 / 63, 1025^3 27.6 / 31.4, but 4097^3 1021 / 693)
                if (f32 && i >= kSplit && (p.fringe_m != 0 || p.fringe_n != 0) && (sl > 1 || blocks <= kComputeUnits)) continue;
                // (an unsliced triangular operand runs below its estimate, most of its sums being shorter: TRMM FP16 3000 x 300 33 us, 38 in slices)
                // (FP32 triangles: two slices run 10-25 % above their estimate, us unsliced on the FP32 pipes / in two slices: 3264 x 2941 271 / 303, 2688 x
                // 2803 178 / 205, 3345 x 3792 372 / 407, 954 x 728 18.9 / 22.4, 785 x 1056 23.5 / 25.6; more slices on the FP32 pipes for more than 7 %)
                const double sliced = narrowed ? 1.25 : (f32 && triangle ? (sl == 2 ? 1.2 : (i < kSplit ? 1.07 : 1.0)) : 1.0);
                const double time = sl == 1 ? unsliced : estimate(i, sl) * sliced;
                if (sl > 1 && static_cast<size_t>(sl) * p.m * p.n * sizeof(float) > workspace_bytes) continue;
                if (ranked[i].slices == 0 || time < ranked[i].time) ranked[i] = Ranked{sl, time};
            }
        }
        // The shared-sum kernel among them, in the same way (4 % rms): (64, 64, 256) both along k 3.2 us, 64 x 64 tiles
        // 3.7, but (704, 128, 64) neither along k 4.7, 3.6
        if (few_blocks && whole_short) {
            double best_us = 1.0e30;
            for (int i = 0; i < count; ++i)
                if (ranked[i].slices != 0 && ranked[i].time * 1.0e-6 < best_us) best_us = ranked[i].time * 1.0e-6;
            const double ktile = p.a_trans ? (p.b_trans ? 0.14 : 0.07) : (p.b_trans ? 0.17 : 0.10), first = p.a_trans ? (p.b_trans ? 0.36 : 0.0) : (p.b_trans ? 0.78 : 0.43);
            const double us = 3.0 + first + (p.beta != 0.f ? 0.44 : 0.0) + ktile * static_cast<double>(p.k / 64) + 0.23 * static_cast<double>(blocks32) / kComputeUnits;
            if (1.03 * us < best_us) {
                char name[48];
                snprintf(name, sizeof name, "htiny_32x32_%s", order_tag);
                if (try_pick(table, p, alignment, name, 1, kernel, split)) return;
            }
        }
        for (int attempt = 0; attempt < count; ++attempt) {
            int best = -1;
            for (int i = 0; i < count; ++i)
                if (!tried[i] && ranked[i].slices != 0 && (best < 0 || ranked[i].time < ranked[best].time)) best = i;
            if (best < 0) break;
            const int want = ranked[best].slices;
            const double best_time = ranked[best].time;
            // FP16 products with a triangular C are ranked by the tiles that touch it (us, ranked as all of C / now: 2048^3 25 / 17,
            // 2560^3 36 / 24, 3584 x 1024 33 / 20, 4096^3 84 both).  A triangular operand (unequal K ranges) is ranked like
            // the general problem (TRMM, us, before the kernels with three and four stages / with them: 1536 25.5 / 21.4, 2048 30.5 /
            // 26.9, 2304 40.9 / 36.1, 2560 45.1 / 39.5, 2816 52.6 / 44.3, 3072 x 1024 40.5 / 33.6, 3328 60.2 / 61.4, 4096 89.2 / 89.7), with one
            // measured exception: when the 256 x 256 direct-to-LDS grid leaves compute units idle anyway, the 128 x 128 tiles
            // balance the unequal work better (3072: 55.5 against 65.4 us)
            if (!f32 && !any_family && p.shape != MG_SHAPE_GENERAL && !triangle && best == 0 && !tried[2] &&
                ceil_div(p.m, 256) * ceil_div(p.n, 256) <= (kComputeUnits * 3) / 4)
                best = 2;
            tried[best] = true;
            const TileChoice &tc = tiles[best];
            if (thin && want == 1 && few_blocks) {       // (no room for slices, or nothing to gain from them)
                char name[48];
                snprintf(name, sizeof name, "%ctiny_32x32_%s", f32 ? 's' : 'h', order_tag);
                if (try_pick(table, p, alignment, name, 1, kernel, split)) return;
            }
            // a factor whose last slice would be empty is illegal: take the next smaller one
            for (int w = want; w >= 1; --w)
                if (try_mfma(table, p, alignment, tc.tag, w, kernel, split)) {
                    if (estimated_us != nullptr) *estimated_us = best_time * 1.0e-6;
                    return;
                }
        }
    }
    if (thin) {                                          // (FP16 of fewer than eight rows that no ranked tile takes: 4 x 30797 x 5268 1267 / 104 us)
        char name[48];
        snprintf(name, sizeof name, "%ctiny_32x32_%s", f32 ? 's' : 'h', order_tag);
        if (try_pick(table, p, alignment, name, 1, kernel, split)) return;
    }
    try_pick(table, p, alignment, f32 ? "direct_f32_64x64x16" : "direct_f16_64x64x16", 1, kernel, split);
}

namespace {

// Estimated us of an FP32 batched call on the kernels of batched_lines.hip (team: 1, 4, 8 wavefronts per instance) and on the tiles of batched_tile.hip that
// select_batched takes otherwise (32 x 32, 32 x 64, 64 x 64), fitted to 22000 random calls (1 to 700 in an extent, 1 to 200000 instances, both routes in one
// build), 7 to 8 % rms.  Whether the device's scalars add the old C of a generic call the host does not know: counted as half of them.
struct BatchedTerms {
    double per_cu, far_mb, c, old_c, bytes, steps, blocks;
    bool generic, stray;

    explicit BatchedTerms(const BatchedProblem &p)
    {
        per_cu = static_cast<double>(p.batch) / kComputeUnits;                                    // instances
        bytes = 4.0 * static_cast<double>(p.m * p.k + p.k * p.n + p.m * p.n);                     // of an instance
        far_mb = static_cast<double>(p.batch) * bytes * 1.0e-6 - 250.0;                           // beyond the last-level cache
        if (far_mb < 0.0) far_mb = 0.0;
        old_c = p.strided ? (p.beta != 0.f ? 1.0 : 0.0) : 0.5;
        c = per_cu * static_cast<double>(p.m * p.n) * 1.0e-3;
        steps = static_cast<double>(ceil_div(p.k, 16));
        blocks = static_cast<double>(ceil_div(p.m, 16) * ceil_div(p.n, 16));
        generic = !p.strided;
        stray = p.m % 4 != 0;                                                                     // columns of C end inside a piece
    }
};

double batched_lines_us(const BatchedProblem &p, int team, const LinesShape &shape)
{
    // per turn of the resident teams: a unit of blocks, its K-steps, its stray ends, an instance's offsets, columns of C shorter than a piece;
    // per compute unit: an instance, K-steps of blocks, 100 pieces of a generic instance, 1000 old elements of C, 10000 bytes
    struct Cost {
        double fixed, unit, instance, block_step, far_mb, stray_unit, generic_turn, generic_pieces, old_c, short_unit, unit_step, bytes;
    };
    static const Cost costs[3] = {{3.65, 0.586, 0.0535, 0.00476, 0.0673, 0.0713, 0.236, 0.00324, 0.0919, 0.201, 0.0796, 0.208},
                                  {3.79, 0.566, 0.172, 0.0113, 0.0446, 0.0843, 0.23, 0.0, 0.0961, 0.349, 0.0804, 0.16},
                                  {4.02, 0.585, 0.391, 0.0129, 0.0336, 0.101, 0.246, 0.0, 0.0985, 0.436, 0.0875, 0.135}};
    const Cost &k = costs[team == 1 ? 0 : (team == 4 ? 1 : 2)];
    const BatchedTerms t(p);
    const int64_t rows = ceil_div(p.m, 16), cols = ceil_div(p.n, 16), groups = ceil_div(rows, 2);
    const int64_t rows_per_group = groups * cols < team ? 1 : ceil_div(rows, groups);            // as the kernel deals its units out
    const double units = static_cast<double>(ceil_div(ceil_div(rows, rows_per_group) * cols, team)), turns = static_cast<double>(ceil_div(p.batch, shape.resident));
    double us = k.fixed + turns * units * (k.unit + k.unit_step * static_cast<double>(rows_per_group) * t.steps);
    if (t.stray) us += turns * units * k.stray_unit;
    if (p.m < 4) us += turns * units * t.old_c * k.short_unit;
    us += t.per_cu * (k.instance + k.block_step * t.blocks * t.steps + k.bytes * t.bytes * 1.0e-4) + k.old_c * t.old_c * t.c + k.far_mb * t.far_mb;
    if (t.generic) us += turns * k.generic_turn + t.per_cu * k.generic_pieces * static_cast<double>(shape.pieces) * 1.0e-2;
    return us;
}

double batched_tile_us(const BatchedProblem &p, int64_t tm, int64_t tn)
{
    // a chunk of the sum; turns of four work-groups per compute unit, and of the columns of blocks that a wavefront has in them; per compute unit: a tile,
    // K-steps of blocks, chunks with lines that end inside a piece, 1000 old elements of C, 10000 bytes
    struct Cost {
        double fixed, chunk, turn, tile, block_step, far_mb, stray_old, stray_chunk, old_c, turn_col, turn_col_step, chunk_col, bytes;
    };
    static const Cost costs[3] = {{3.25, 0.44, 0.608, 0.0, 0.00639, 0.0396, 0.54, 0.00727, 0.238, 0.0, 0.118, 0.164, 0.106},
                                  {3.63, 0.0548, 0.0, 0.298, 0.0112, 0.0101, 0.461, 0.00889, 0.0786, 0.146, 0.105, 0.114, 0.128},
                                  {3.39, 0.26, 0.0, 0.324, 0.0117, 0.0261, 0.579, 0.0212, 0.102, 0.394, 0.0817, 0.174, 0.158}};
    const Cost &k = costs[tn == 32 ? 0 : (tm == 32 ? 1 : 2)];
    const BatchedTerms t(p);
    const int64_t tiles = ceil_div(p.m, tm) * ceil_div(p.n, tn), blocks_n = ceil_div(p.n, 16);
    const double chunks = static_cast<double>(ceil_div(p.k, 32)), turns = static_cast<double>(ceil_div(p.batch * tiles, 4 * kComputeUnits));
    const double cols = (tn == 32 ? blocks_n : ceil_div(blocks_n, 2)) > 1 ? 2.0 : 1.0;
    const double stray_lines = ((p.a_trans ? p.k : p.m) % 4 != 0 ? 1.0 : 0.0) + ((p.b_trans ? p.n : p.k) % 4 != 0 ? 1.0 : 0.0);
    double us = k.fixed + chunks * (k.chunk + k.chunk_col * cols) + turns * (k.turn + cols * (k.turn_col + k.turn_col_step * t.steps));
    us += t.per_cu * (static_cast<double>(tiles) * (k.tile + k.stray_chunk * stray_lines * chunks) + k.block_step * t.blocks * t.steps + k.bytes * t.bytes * 1.0e-4);
    return us + (t.stray ? k.stray_old * t.old_c : 0.0) + k.old_c * t.old_c * t.c + k.far_mb * t.far_mb;
}

}  // namespace

int32_t select_batched(const std::vector<KernelEntry> &table, const BatchedProblem &p)
{
    // One wavefront per instance while the instance fits the register blocks (<= 32 in every extent); with more 16^3
    // instances than wavefronts fit on the chip at once (256 compute units x 32), two per wavefront: measured 7.0 -> 6.4 us
    // (FP32) and 5.3 -> 4.7 us (FP16) for 10000 instances, no gain from four, a loss below ~4000 instances
    // (FP32 instances smaller than 16^3 take the bounds-checked flavour, which gains nothing from the second
    // instance: 10000 x 8^3 5.5 us one per wavefront, 5.9 us two)
    const bool whole16 = p.m == 16 && p.n == 16 && p.k == 16;
    // FP32 instances whose operands no longer fit the last-level cache by a wide margin (HBM-real calls) are faster one
    // per wavefront again; 16^3, us one / two per wavefront: 120000 instances (379 MB of operands) 82.3 / 79.5, 140000
    // (442 MB) 101.2 / 107.9, 160000 117.3 / 131.6, 200000 (631 MB) 145.6 / 162.7.  FP16 stays with two (320000 instances,
    // 505 MB: 141.0 / 122.5).
    const double operand_bytes = static_cast<double>(p.batch) * static_cast<double>(p.m * p.k + p.k * p.n + p.m * p.n) * (p.dtype == MG_F32 ? 4.0 : 2.0);
    const bool streams_from_hbm = p.dtype == MG_F32 && operand_bytes > 410.0e6;
    const bool pairs = p.batch >= 32 * kComputeUnits && !streams_from_hbm && (p.dtype != MG_F32 || whole16);
    const char *prefix = p.dtype == MG_F32 ? "" : "h";
    const char *contig = p.a_trans ? (p.b_trans ? "kn" : "kk") : (p.b_trans ? "mn" : "mk");
    // whole 64^3 instances with A along m and B along k: the kernels whose lanes are rows of C ask for A, B and C in whole
    // adjacent columns (1 KB runs instead of 64-byte ones): FP32 10000 instances 155 -> 116 us, FP16 85 -> 49 us.  FP32 with
    // four wavefronts per instance (a quarter of the columns each) is never slower than one and faster for few
    // instances (us, one / four: 200 instances 8.9 / 6.0, 500: 9.8 / 7.8, 1000: 14.4 / 14.2, 4000: 43.3 / 41.6, 10000: 116.6 / 116.3)
    for (const char *name : {"batched_rows_64w4_mk_full", "batched_rows_64_mk_full", "hbatched_rows_64_mk_full"}) {
        const int32_t id = find(table, name);
        if (id >= 0 && table[id].legal_batched(p)) return id;
    }
    auto take = [&](const char *tag, const char *suffix) {
        char name[96];
        snprintf(name, sizeof name, "%s%s_%s%s", prefix, tag, contig, suffix);
        const int32_t id = find(table, name);
        return id >= 0 && table[id].legal_batched(p) ? id : -1;
    };
    // Whole instances through LDS (batched_lines.hip), one, four or eight wavefronts each.  From 420 random calls (8 to 160 in an extent, 1 to 20000
    // instances, every kernel forced):
    //   * up to 32 in every extent only FP16 that is not along k on both sides, whose register blocks take two bytes per load (us, those / these: 27 x 28 x 30,
    //     7000 instances 17.0 / 9.6; 26^3 along k, 1752 instances 4.7 / 5.2; FP32 23^3, 1200 instances 5.2 / 6.5);
    //   * FP32 of 41 to 64 rows and columns fills the 64 x 64 tile (48^3, 14200 instances 81 / 86; 35^3, 6415 instances 45 / 37), FP16 of 64 x 64 too
    //     (1702 instances of 64^3 10.0 / 11.6);
    //   * whole 32^3 with A along m and B along k has unchecked register blocks (FP16, 1800 instances 4.4 / 5.2);
    //   * FP32 sums of more than 80 terms, and of more than 48 on 17 to 33 rows or columns, stay with the tiles in large batches (48 x 32 x 135, 3926
    //     instances 39 / 51; 19 x 23 x 56, 15100 instances 44 / 55; 72 x 12 x 52, 9800 instances 72 / 48);
    //   * a handful of large instances is cut into tiles below (20 of 76^3 FP32 5.6 / 8.0);
    //   * one wavefront each where there are enough instances for the chip and few blocks of 16 x 16 in them (45 x 37 x 16, 9600 FP16 instances: old 41,
    //     one wavefront 21.5, four 24.8; 126 x 28 x 12, 15300 instances 100 / 58 / 50);
    //   * four where a compute unit has several instances, else eight (74^3, 485 instances: old 11.7, four 7.3, eight 6.8).
    const auto lines = [&]() -> int32_t {
        const int64_t most = p.m > p.n ? (p.m > p.k ? p.m : p.k) : (p.n > p.k ? p.n : p.k), blocks = ceil_div(p.m, 16) * ceil_div(p.n, 16);
        const bool f32 = p.dtype == MG_F32;
        if (most <= 16 || (most <= 32 && (f32 || (p.a_trans && !p.b_trans)))) return -1;
        if (most <= 20 && p.a_trans) return -1;                       // (6900 x 18^3, A along k, B along n 7.3 / 8.8)
        // (8000 x 17^3 9.0 / 10.9; 23 calls 1.06)
        if (most <= 17 && !p.a_trans && !p.b_trans && p.batch >= kComputeUnits) return -1;
        if (p.batch < 130 && blocks > 12) return -1;
        if (f32 && p.m > 40 && p.m <= 64 && p.n > 40 && p.n <= 64 && p.k > 16) return -1;
        if (!f32 && p.m == 64 && p.n == 64) return -1;
        // (of a generic batch, whose instances may lie anywhere, whole pieces that fill most of a tile and its chunk: 48^3 and 56^3, 130 calls of all orders 1.14 times
        // as long, 9500 x 48^3 1.23, 16610 x 56^3 63 / 86 us; strided 0.97)
        if (!f32 && !p.strided && p.batch >= 1000 && p.m > 40 && p.m <= 64 && p.n > 40 && p.n <= 64 && p.k > 32 && p.k <= 64 && p.m % 8 == 0 && p.n % 8 == 0 && p.k % 8 == 0) return -1;
        if (!f32 && take("batched_wave_32", "_full") >= 0) return -1;
        const int64_t thin = p.m < p.n ? p.m : p.n;
        if (f32 && p.batch >= 1000 && (p.k > 80 || (p.k > 48 && thin > 16 && thin <= 33))) return -1;
        if (p.batch >= 1000 && blocks <= (f32 ? 6 : 12)) {
            const int32_t id = take("batched_lines_w1", "");
            // (FP32 lines along the rows of 24 x 40 x 24: two work-groups' LDS per compute unit, 5900 instances 20.9 / 28.4)
            if (id >= 0 && !(f32 && blocks > 4 && p.k > 16)) return id;
        }
        if (blocks < 2 && p.k > 64 && p.batch >= 1000) return -1;
        const int32_t four = take("batched_lines_w4", "");
        if (four >= 0 && p.batch >= 256) return four;
        const int32_t eight = blocks >= 6 ? take("batched_lines_w8", "") : -1;
        return eight >= 0 ? eight : four;
    };
    // (FP32 calls that they are estimated to lose stay below, with the estimates' error on the side of these kernels.  By the lines above alone 15 % of the FP32 calls
    // were more than 5 % slower than below, up to 1.7 times: 2982 x (32, 16, 40) 8.9 / 12.6, 2855 x (24, 104, 48) 27 / 39, 76 x (7, 152, 6) 4.6 / 6.1; with the
    // estimates 3 %, up to 1.27, and 0.7 % give up more than 5 %.  Fitted to half of the calls, counted on the others.  FP16: 3 %, without.)
    {
        const bool small = p.m <= 32 && p.n <= 32, narrow = ceil_div(p.m, 32) % 2 != 0;
        const int32_t id = lines();
        LinesShape shape;
        const int team = id >= 0 ? table[id].cfg.waves_n : 0;
        // (from 33 rows and columns the tiles' estimates are 5 to 10 % too low, mostly with beta: of 770 calls of up to 96 rows and columns and more than 32 terms they sent 78 to
        // slower tiles and 22 to faster ones, 5415 x 38^3 with beta 31.5 us / 34.6, 7331 x (63, 68, 68) 119 / 155, and of 305 strided ones with beta of any larger size 12 and 2)
        const int64_t thin = p.m < p.n ? p.m : p.n, wide = p.m < p.n ? p.n : p.m;
        const bool stands = thin > 32 && ((wide <= 96 && p.k > 32) || (p.strided && p.beta != 0.f));
        if (id >= 0 && (p.dtype != MG_F32 || stands || !batched_lines_shape(p, team, &shape) ||
                        batched_lines_us(p, team, shape) < 1.02 * batched_tile_us(p, small || narrow ? 32 : 64, small ? 32 : 64))) return id;
    }
    // (FP32 instances that fill the 32 x 32 block and stream from memory lose more to the one-wavefront kernel's 4-byte and
    // unaligned requests than its shorter latency chain gains: 31^3, four operand orders, LDS-staged / one wavefront: 10000
    // instances 28 / 35 us, 1000 instances 6.6 / 5.8 us; 28^3 24.5 / 21-25 us, FP16 31^3 26-34 / 20-24 us; whole 32^3 with A along m
    // and B along k 25.7 / 24.6 us)
    const bool filled = p.dtype == MG_F32 && p.m > 28 && p.n > 28 && p.k > 28 && p.m <= 32 && p.n <= 32 && p.k <= 32 && p.batch >= 4096;
    for (const char *tag : {pairs ? "batched_wave_16x2" : "batched_wave_16", "batched_wave_32"}) {
        int32_t id = take(tag, "_full");
        if (id < 0 && !filled) id = take(tag, "");
        if (id >= 0) return id;
    }
    // LDS-staged tiles.  A longer sum with at most 32 x 32 outputs: one wavefront per instance (24 x 16 x 40, 6300 FP32
    // instances: 13 us against 17 us with four).  Else four wavefronts on a 64 x 64 tile, or on 32 x 64 where that pads less: FP32
    // 93^3 (856 instances) 31 us on 32 x 64, 39 us on 64 x 64; 64^3 (5000) 73 / 69 us; 99^3 201 / 191 us; FP16 19 x 80 x 144
    // (2100) 23 / 25 us, 81^3 (800) 17 / 15 us, 37^3 (2300) 15 / 12 us: FP16, whose loads are the smaller part, only below 33 rows.
    // (96 x 64, 128 x 64 and 128 x 128 tiles, whose teams leave fewer work-groups to overlap: 10-60 % slower on most of these.)
    const bool thin = p.dtype == MG_F32 ? ceil_div(p.m, 32) % 2 != 0 : p.m <= 32;
    if (p.m <= 32 && p.n <= 32) {
        const int32_t id = take("batched_tile_32x32", "");
        if (id >= 0) return id;
    }
    for (const char *tag : {thin ? "batched_tile_32x64" : "batched_tile_64x64", "batched_tile_64x64"}) {
        const int32_t id = take(tag, "");
        if (id >= 0) return id;
    }
    return -1;
}

}  // namespace mg
