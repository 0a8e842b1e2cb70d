// FP16 tiles for operands whose rows start at any element (mfma_any_kernel.h).  Against the best of the register-staged tiles with checks, any slices,
// us: 1500^3 20.2 / 17.9, 1501^3 (odd rows) 26.9 / 22.5, 2051^3 46.4 / 34.1, (533, 696, 991) 11.3 / 9.6, (143, 5204, 475) with beta 8.7 / 7.5; geometric mean
// over 700 products of 64 to 8192 terms 0.76.  Their code is 6 to 10 KB where those have 20 to 27.
//   * 64 x 64 and 128 x 64: four K-tiles in flight, 0.25 and 0.33 us per K-tile and turn (64 x 64 direct-to-LDS, rows on 16 bytes: 0.16);
//   * 128 x 128: four as well (162 registers, one work-group per compute unit); two K-tiles together every second one, so that the line that two K-tiles
//     of a row share is still in the L1, 1501^3 26.2 instead of 24.7 us: the bursts wait for each other;
//   * 192 x 128 and 256 x 128: two K-tiles in flight, 2051^3 34.7 and 38.3.
#include "mfma_dma_host.h"
#include "mfma_any_kernel.h"
namespace mg {
namespace {
template <int BM, int BN, int WM, int WN, bool AK, bool BKC, int DEPTH> struct MfmaAnyConfig {
    using Checked = MfmaConfig<_Float16, BM, BN, 64, WM, WN, AK, BKC, true>;   // same legality and split-K rules
    static constexpr int NT = WM * WN * 64;
    static constexpr int LDS = 2 * (BM + BN) * 128 > any_result_bytes<BM, BN>() ? 2 * (BM + BN) * 128 : any_result_bytes<BM, BN>();
    static_assert(LDS <= 160 * 1024, "LDS of a compute unit");

    static bool legal(const Problem &p, int split, int64_t alignment)
    {
        // (loads of 16 bytes that end with a line or run seven elements into the next one)
        if (p.k < 8 || p.m < 8 || p.n < 8) return false;
        // (a grid of the wanted tiles of a triangle wants a square C)
        if (p.shape >= MG_SHAPE_C_LOWER && p.m != p.n) return false;
        return Checked::legal(p, split, alignment);
    }
    static hipError_t launch(const Problem &p, int split)
    {
        static bool attr_set = false;   // raising the dynamic LDS limit is idempotent; races are harmless
        return launch_tile_kernel<_Float16>(hgemm_any_kernel<BM, BN, WM, WN, AK, BKC, DEPTH>, &attr_set, LDS, NT, BM, BN,
                                            Checked::k_per_split(p, split), p, split, 0, BM == BN);
    }
    static KernelEntry entry(const char *name)
    {
        KernelEntry e = Checked::entry(name, launch);
        e.cfg.lds_bytes = LDS;
        e.legal = legal;
        return e;
    }
};
}  // namespace
#define MG_ANY(tag, BM, BN, WM, WN, DEPTH)                                                  \
    table.push_back(MfmaAnyConfig<BM, BN, WM, WN, true, true, DEPTH>::entry(tag "_kk"));   \
    table.push_back(MfmaAnyConfig<BM, BN, WM, WN, false, true, DEPTH>::entry(tag "_mk"));  \
    table.push_back(MfmaAnyConfig<BM, BN, WM, WN, true, false, DEPTH>::entry(tag "_kn"));  \
    table.push_back(MfmaAnyConfig<BM, BN, WM, WN, false, false, DEPTH>::entry(tag "_mn"));
void register_hany16(std::vector<KernelEntry> &table)
{
    MG_ANY("hany16_256x128x64_w4x2", 256, 128, 4, 2, 2)
    MG_ANY("hany16_192x128x64_w2x4", 192, 128, 2, 4, 2)
    MG_ANY("hany16_128x128x64_w2x4", 128, 128, 2, 4, 4)
    MG_ANY("hany16_128x64x64_w4x2", 128, 64, 4, 2, 4)
    MG_ANY("hany16_64x64x64_w2x2", 64, 64, 2, 2, 4)
}
}  // namespace mg
