// FP32 on the bf16 matrix pipes, tile 256 x 128 x 32, 4 x 2 wavefronts, 1 K-tile in flight.
#include "mfma_split_host.h"
namespace mg {
void register_ssplit_256x128x32_w4x2(std::vector<KernelEntry> &table)
{
    MG_SPLIT_REGISTER(table, "ssplit_256x128x32_w4x2", 256, 128, 4, 2, 1)
}
}  // namespace mg
