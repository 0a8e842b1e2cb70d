// FP32 on the bf16 matrix pipes, 64 x 64 tiles, eight wavefronts that share the sum.
#include "mfma_split_host.h"
namespace mg {
void register_ssplit_slices_64x64(std::vector<KernelEntry> &table)
{
    table.push_back(SplitSlicesConfig<false, true, false>::entry("ssplit_slices_64x64_mk"));
    table.push_back(SplitSlicesConfig<true, true, false>::entry("ssplit_slices_64x64_kk"));
    table.push_back(SplitSlicesConfig<false, false, false>::entry("ssplit_slices_64x64_mn"));
    table.push_back(SplitSlicesConfig<true, false, false>::entry("ssplit_slices_64x64_kn"));
    table.push_back(SplitSlicesConfig<false, true, true>::entry("ssplit_slices_64x64_mk_edge"));
    table.push_back(SplitSlicesConfig<true, true, true>::entry("ssplit_slices_64x64_kk_edge"));
    table.push_back(SplitSlicesConfig<false, false, true>::entry("ssplit_slices_64x64_mn_edge"));
    table.push_back(SplitSlicesConfig<true, false, true>::entry("ssplit_slices_64x64_kn_edge"));
}
}  // namespace mg
