// FP32 on the bf16 matrix pipes, tile 128 x 128 x 32, 2 x 4 wavefronts, 1 K-tile in flight.
#include "mfma_split_host.h"
namespace mg {
void register_ssplit_128x128x32_w2x4(std::vector<KernelEntry> &table)
{
    MG_SPLIT_REGISTER(table, "ssplit_128x128x32_w2x4", 128, 128, 2, 4, 1)
}
}  // namespace mg
