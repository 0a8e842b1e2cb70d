// Host-side rules and registration helpers of the FP32 kernels on the bf16 matrix pipes.
#pragma once

#include "mfma_host.h"
#include "mfma_split_kernel.h"

namespace mg {

template <int BM, int BN, int WM, int WN, bool AK, bool BKC, bool EDGE, int DEPTH> struct SplitConfig {
    using Plain = MfmaConfig<float, BM, BN, 32, WM, WN, AK, BKC, EDGE>;      // the same tile's rules
    static constexpr int NT = WM * WN * 64;
    static constexpr int STAGES_LDS = 2 * 3 * (BM + BN) * 64;
    static constexpr int LDS = STAGES_LDS > Plain::EPILOGUE_LDS ? STAGES_LDS : Plain::EPILOGUE_LDS;

    static hipError_t launch(const Problem &p, int split)
    {
        static bool attr_set = false;   // raising the dynamic LDS limit is idempotent; races are harmless
        return launch_tile_kernel<float>(mfma_split_kernel<BM, BN, WM, WN, AK, BKC, EDGE, DEPTH>, &attr_set, LDS, NT, BM, BN,
                                         Plain::k_per_split(p, split), p, split, EDGE ? Plain::fringe_groups(p) : 0);
    }
    static KernelEntry entry(const char *name)
    {
        KernelEntry e = Plain::entry(name, launch);
        e.cfg.lds_bytes = LDS;
        return e;
    }
};

#define MG_SPLIT_REGISTER(table, tag, BM, BN, WM, WN, DEPTH)                                          \
    table.push_back(SplitConfig<BM, BN, WM, WN, false, true, false, DEPTH>::entry(tag "_mk"));        \
    table.push_back(SplitConfig<BM, BN, WM, WN, true, true, false, DEPTH>::entry(tag "_kk"));         \
    table.push_back(SplitConfig<BM, BN, WM, WN, false, false, false, DEPTH>::entry(tag "_mn"));       \
    table.push_back(SplitConfig<BM, BN, WM, WN, true, false, false, DEPTH>::entry(tag "_kn"));        \
    table.push_back(SplitConfig<BM, BN, WM, WN, false, true, true, DEPTH>::entry(tag "_mk_edge"));    \
    table.push_back(SplitConfig<BM, BN, WM, WN, true, true, true, DEPTH>::entry(tag "_kk_edge"));     \
    table.push_back(SplitConfig<BM, BN, WM, WN, false, false, true, DEPTH>::entry(tag "_mn_edge"));   \
    table.push_back(SplitConfig<BM, BN, WM, WN, true, false, true, DEPTH>::entry(tag "_kn_edge"));

}  // namespace mg
